"""Exact mode and the small table on rows at the edges of the tiers: a wave's table, the two
workgroup sizes, and the global table; few keys, many keys and every entry its own key, and
user-set tier bounds.  Sweeps and refinement against the CPU oracle.  Run on an MI355X only."""
import numpy as np
import pytest

import oracle
from test_gpu_rows import hub_graph, mg  # noqa: F401 (the library's fixture)

pytestmark = pytest.mark.gpu

DEGREES = [33, 63, 64, 65, 127, 128, 129, 192, 255, 256, 257, 511, 512, 513, 768, 1022, 1023, 1024, 1025, 2047, 2048,
           2049, 4095, 4096, 4097, 256]


@pytest.mark.parametrize("tiers", [{}, dict(exact_small=1, exact_lds=40, exact_lds_big=600),
                                   dict(exact_small=300, exact_lds=512, exact_lds_big=1024),
                                   dict(exact_lds=100, exact_lds_big=100)])
@pytest.mark.parametrize("mode,k", [(0, 8), (5, 7), (5, 20000)])
def test_exact_tiers(mg, mode, k, tiers):  # noqa: F811
    import torch
    g = hub_graph(DEGREES, 4500, 6, seed=k)
    dg = mg.to_device(g)
    rng = np.random.default_rng(k)
    for groups in (2, 90, g.n):
        C = rng.integers(0, groups, size=g.n).astype(np.int32)
        tC = torch.from_numpy(C).to("cuda")
        for algo, oalgo in ((mg.ALGO_LPA, oracle.ALGO_LPA), (mg.ALGO_LOUVAIN, oracle.ALGO_MOVE)):
            Cn, gain, ctr = mg.move_sweep(dg, algo, tC, 0, mode=mode, k=k, **tiers)
            eC, eg = oracle.move_sweep(g, oalgo, C, mode=mode, k=k, direction=0)
            assert np.array_equal(Cn.cpu().numpy(), eC), (groups, algo)
            assert ctr[0] == int((eC != C).sum())
            if algo == mg.ALGO_LOUVAIN:
                assert np.array_equal(gain.cpu().numpy(), eg)
        R = mg.refine(dg, tC, mode=mode, k=k, **tiers)
        assert np.array_equal(R.cpu().numpy(), oracle.refine(g, C, mode=mode, k=k)), groups
