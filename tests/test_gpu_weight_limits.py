"""Total weights up to the largest accepted, 2^31 - 1, with vertices and communities that
hold most of it: the gains' 32-bit factors at their limits.  Against the CPU oracle's
64-bit arithmetic, bit for bit.  Run on an MI355X only."""
import numpy as np
import pytest

import oracle
from paper_2411_02268_amd import synth
from test_gpu_rows import mg  # noqa: F401 (the library's fixture)

pytestmark = pytest.mark.gpu

TOP = (1 << 31) - 1


def heavy_graph(heavy, seed):
    """Hubs over all row classes with weights 1 .. 9 and a few edges that bring the total to
    2^31 - 1: between two hubs, between a hub and leaves, or a self-loop."""
    rng = np.random.default_rng(seed)
    degrees, leaves = [2, 5, 14, 30, 33, 60, 130, 300, 700], 900
    pairs = {}
    for h, deg in enumerate(degrees):
        for v in rng.choice(leaves, size=deg, replace=False):
            pairs[(int(v), leaves + h)] = int(rng.integers(1, 10))
    for v in range(0, leaves - 1, 2):
        pairs[(v, v + 1)] = 1
    left = TOP - 1 - 2 * sum(pairs.values())
    loops = {}
    if heavy == "hubs":
        pairs[(leaves + 7, leaves + 8)] = left // 2
        loops[3] = 1 + left % 2
    elif heavy == "leaves":
        mine = [p for p in pairs if p[1] == leaves + 6][:4]
        for p in mine:
            pairs[p] += left // 8
        loops[leaves + 6] = TOP - 2 * sum(pairs.values())
    else:
        loops[leaves + 8] = left + 1
    edges, ws = list(pairs), list(pairs.values())
    g = synth.from_edges(leaves + len(degrees), edges, weights=ws, self_loops=loops)
    assert int(g.weights.astype(np.int64).sum()) == TOP
    return g


@pytest.mark.parametrize("heavy", ["hubs", "leaves", "loop"])
@pytest.mark.parametrize("kw", [{"mode": 1, "k": 8}, {"mode": 1, "k": 16, "short_rows": 2}, {"mode": 2, "k": 4},
                                {"mode": 3, "k": 2}, {"mode": 1, "k": 64}, {"mode": 2, "k": 128}, {"mode": 0, "k": 8},
                                {"mode": 0, "k": 8, "exact_small": 1, "exact_lds": 1, "exact_lds_big": 1},
                                {"mode": 5, "k": 50}])
def test_weight_limits(mg, kw, heavy):  # noqa: F811
    import torch
    okw = {x: kw[x] for x in ("mode", "k")}
    for seed in range(3):
        g = heavy_graph(heavy, seed)
        dg = mg.to_device(g)
        rng = np.random.default_rng(seed)
        for groups in (2, 30, 0):
            C = rng.integers(0, groups, size=g.n).astype(np.int32) if groups else np.arange(g.n, dtype=np.int32)
            tC = torch.from_numpy(C).to("cuda")
            for algo, oalgo in ((mg.ALGO_LPA, oracle.ALGO_LPA), (mg.ALGO_LOUVAIN, oracle.ALGO_MOVE)):
                Cn, gain, _ = mg.move_sweep(dg, algo, tC, 0, **kw)
                eC, eg = oracle.move_sweep(g, oalgo, C, direction=0, **okw)
                assert np.array_equal(Cn.cpu().numpy(), eC), (groups, algo)
                if algo == mg.ALGO_LOUVAIN:
                    assert np.array_equal(gain.cpu().numpy(), eg), groups
            R = mg.refine(dg, tC, **kw)
            assert np.array_equal(R.cpu().numpy(), oracle.refine(g, C, **okw)), groups
        for algo in ("louvain", "leiden"):
            lab, _ = getattr(mg, algo)(dg, **kw, **({"k_aggregate": 8} if kw["mode"] == 5 else {}))
            okw2 = {**okw, **({"k_aggregate": 8} if kw["mode"] == 5 else {})}
            assert np.array_equal(lab.cpu().numpy(), getattr(oracle, algo)(g, **okw2)[0]), algo
