"""Sketches of 32 to 256 slots at the edges of the wave kernels: as many different keys as
slots and one more, batches of 64 items, chunks that are no multiple of a batch, rows on
both sides of the split, and merge trees on both sides of the levels that have a launch of
their own.  Sweeps, refinement and aggregation against the CPU oracle, bit for bit.  Run on
an MI355X only."""
import numpy as np
import pytest

import oracle
from test_gpu_rows import MODES, hub_graph, mg  # noqa: F401 (the library's fixture)

pytestmark = pytest.mark.gpu

EDGES = {  # chunk length -> hub degrees
    8: [33, 64, 65, 512, 513, 2040, 2048, 2049, 2056, 4097],
    100: [63, 99, 100, 101, 164, 200, 201, 512, 513, 1000],
    128: [32, 33, 63, 64, 65, 127, 128, 129, 192, 193, 255, 256, 257, 384, 385, 511, 512, 513, 640, 4097],
    600: [96, 97, 320, 321, 599, 600, 601, 1200, 1201],
}


@pytest.mark.parametrize("mode", ["alg1", "uncond", "std"])
@pytest.mark.parametrize("k", [32, 64, 128, 256])
@pytest.mark.parametrize("L", sorted(EDGES))
def test_wave_rows(mg, mode, k, L):  # noqa: F811
    import torch
    g = hub_graph(EDGES[L], 4500, 6, seed=k + L)
    dg = mg.to_device(g)
    kw = {"mode": MODES[mode], "k": k, "chunk_len": L}
    for groups in (k, k + 1, 3 * k, g.n):
        C = (np.arange(g.n) * 7919 % groups).astype(np.int32)
        tC = torch.from_numpy(C).to("cuda")
        for algo, oalgo in ((mg.ALGO_LPA, oracle.ALGO_LPA), (mg.ALGO_LOUVAIN, oracle.ALGO_MOVE)):
            Cn, gain, ctr = mg.move_sweep(dg, algo, tC, 0, **kw)
            eC, eg = oracle.move_sweep(g, oalgo, C, direction=0, **kw)
            assert np.array_equal(Cn.cpu().numpy(), eC), (groups, algo)
            assert ctr[0] == int((eC != C).sum())
            if algo == mg.ALGO_LOUVAIN:
                assert np.array_equal(gain.cpu().numpy(), eg)
        R = mg.refine(dg, tC, **kw)
        assert np.array_equal(R.cpu().numpy(), oracle.refine(g, C, **kw)), groups


@pytest.mark.parametrize("mode", ["alg1", "uncond", "std"])
@pytest.mark.parametrize("k", [32, 64, 128, 256])
@pytest.mark.parametrize("L", sorted(EDGES))
def test_wave_aggregation(mg, mode, k, L):  # noqa: F811
    import torch
    g = hub_graph(EDGES[L], 4500, 6, seed=k + L)
    dg = mg.to_device(g)
    for groups in (k + 1, 3 * k, 1500):
        D = (np.arange(g.n) * 7919 % groups).astype(np.int32)
        D[-len(EDGES[L]):] = groups + np.arange(len(EDGES[L]))  # each hub alone
        m = int(D.max()) + 1
        got = mg.aggregate(dg, torch.from_numpy(D).to("cuda"), m, mode=MODES[mode], k=k, chunk_len=L)
        want = oracle.aggregate(g, D, m, mode=MODES[mode], k=k, chunk_len=L)
        for a, b in zip(got, (want.offsets, want.indices, want.weights)):
            assert np.array_equal(a, b), groups
