"""Row lengths at the edges of the main sweep kernel's tiles: a light row's 16- and
32-entry loads, a chunk's 32-entry windows and 128-entry limit, a wave's 16 and a
workgroup's 64 chunks, and a row that ends with the arrays.  Sweeps and refinement
against the CPU oracle, bit for bit.  Run on an MI355X only."""
import numpy as np
import pytest

import oracle
from paper_2411_02268_amd import synth

pytestmark = pytest.mark.gpu

MODES = {"alg1": 1, "uncond": 2, "std": 3}


@pytest.fixture(scope="module")
def mg():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_02268_amd as m
    m.lib()
    return m


def hub_graph(degrees, n_leaves, wmax, seed):
    """One hub per degree, each joined to that many distinct leaves; the hubs have the
    highest ids, so the last degree's row ends with the arrays.  Hub 0 has a self-loop."""
    rng = np.random.default_rng(seed)
    edges, ws = [], []
    for h, deg in enumerate(degrees):
        for v in rng.choice(n_leaves, size=deg, replace=False):
            edges.append((int(v), n_leaves + h))
            ws.append(int(rng.integers(1, wmax + 1)))
    return synth.from_edges(n_leaves + len(degrees), edges, weights=ws, self_loops={n_leaves: 3})


EDGES = {  # chunk length -> hub degrees around the kernel's boundaries at that length
    128: [1, 3, 4, 5, 15, 16, 17, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 255, 256, 257, 2047, 2048, 2049,
          4096, 4097, 8191, 8192, 8193, 8250],
    20: [19, 20, 21, 39, 40, 41, 319, 320, 321, 640, 641, 1279, 1280, 1281, 2561],
    700: [32, 33, 64, 65, 699, 700, 701, 1400, 1401, 2801],
}


@pytest.mark.parametrize("mode", ["alg1", "uncond", "std"])
@pytest.mark.parametrize("k", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("L", sorted(EDGES))
def test_row_lengths(mg, mode, k, L):
    import torch
    g = hub_graph(EDGES[L], 9000, 6, seed=k + L)
    dg = mg.to_device(g)
    rng = np.random.default_rng(k)
    for groups in (3, 40, g.n):  # exact sketches, mixed, nearly every entry a key of its own
        C = rng.integers(0, groups, size=g.n).astype(np.int32)
        tC = torch.from_numpy(C).to("cuda")
        for algo, oalgo in ((mg.ALGO_LPA, oracle.ALGO_LPA), (mg.ALGO_LOUVAIN, oracle.ALGO_MOVE)):
            Cn, gain, ctr = mg.move_sweep(dg, algo, tC, 0, mode=MODES[mode], k=k, chunk_len=L)
            eC, eg = oracle.move_sweep(g, oalgo, C, mode=MODES[mode], k=k, chunk_len=L, direction=0)
            assert np.array_equal(Cn.cpu().numpy(), eC), (groups, algo)
            assert ctr[0] == int((eC != C).sum())
            if algo == mg.ALGO_LOUVAIN:
                assert np.array_equal(gain.cpu().numpy(), eg)
                assert ctr[1:] == [int((eg > 0).sum()), int(eg.sum())]
        R = mg.refine(dg, tC, mode=MODES[mode], k=k, chunk_len=L)
        assert np.array_equal(R.cpu().numpy(), oracle.refine(g, C, mode=MODES[mode], k=k, chunk_len=L)), groups


@pytest.mark.parametrize("algo", ["lpa", "louvain"])
def test_counts_of_many_small_graphs(mg, algo):
    """Graphs of a few rows each, so that a wave's rows belong to many graphs, beside
    one whose rows fill several workgroups."""
    graphs = [synth.random_small(3 + s % 29, 0.5, 4, seed=s) for s in range(60)]
    graphs.insert(17, synth.planted_exact(n_comm=8, comm_size=60, seed=5)[0])
    graphs.append(hub_graph([40, 200, 300], 400, 5, seed=9))
    A = mg.ALGO_LPA if algo == "lpa" else mg.ALGO_LOUVAIN
    labs, per, _ = mg.run_batched(A, [mg.to_device(g) for g in graphs], k=8)
    for i, g in enumerate(graphs):
        elab, est = getattr(oracle, algo)(g, k=8)
        assert np.array_equal(labs[i].cpu().numpy(), elab), i
        assert per[i]["iterations"] == est.iterations and per[i]["edges_scanned"] == est.edges_scanned, i


@pytest.mark.parametrize("kw,k", [({"mode": 0}, 8), ({"mode": 0, "exact_small": 64}, 8), ({"mode": 5}, 7),
                                  ({"mode": 5}, 20000), ({"mode": 1, "short_rows": 2}, 16),
                                  ({"mode": 3, "short_rows": 2}, 4), ({"mode": 1}, 32)])
def test_short_row_classes(mg, kw, k):
    """Rows on both sides of each class of the short rows' kernel (1 to 8 lanes per row),
    the last of them ending with the arrays."""
    import torch
    degrees = [1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 40, 64, 65] * 5
    for tail in (1, 2, 4, 5, 31, 32):
        g = hub_graph(degrees + [tail], 500, 6, seed=tail)
        dg = mg.to_device(g)
        rng = np.random.default_rng(k)
        for groups in (3, 40, g.n):
            C = rng.integers(0, groups, size=g.n).astype(np.int32)
            tC = torch.from_numpy(C).to("cuda")
            for algo, oalgo in ((mg.ALGO_LPA, oracle.ALGO_LPA), (mg.ALGO_LOUVAIN, oracle.ALGO_MOVE)):
                Cn, gain, ctr = mg.move_sweep(dg, algo, tC, 0, k=k, **kw)
                eC, eg = oracle.move_sweep(g, oalgo, C, mode=kw["mode"], k=k, direction=0)
                assert np.array_equal(Cn.cpu().numpy(), eC), (tail, groups, algo)
                assert ctr[0] == int((eC != C).sum())
                if algo == mg.ALGO_LOUVAIN:
                    assert np.array_equal(gain.cpu().numpy(), eg)
            R = mg.refine(dg, tC, k=k, **kw)
            assert np.array_equal(R.cpu().numpy(), oracle.refine(g, C, mode=kw["mode"], k=k)), (tail, groups)
