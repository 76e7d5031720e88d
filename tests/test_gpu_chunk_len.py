"""Chunk lengths beyond every stream, up to the largest the parameter holds: one chunk per
row and community, whatever the sum of a position and the length would be.  Against the
CPU oracle, bit for bit.  Run on an MI355X only."""
import numpy as np
import pytest

import oracle
from test_gpu_rows import hub_graph, mg  # noqa: F401 (the library's fixture)

pytestmark = pytest.mark.gpu

LONG = 1 << 40  # the oracle's: any length beyond the rows gives the same


@pytest.mark.parametrize("L", [1 << 31, LONG + 1, 1 << 60, (1 << 61) + 1, 1 << 62, (1 << 63) - 1])
@pytest.mark.parametrize("k,mode", [(8, 1), (16, 3), (64, 1), (128, 1), (256, 2)])
def test_long_chunks(mg, k, mode, L):  # noqa: F811
    import torch
    g = hub_graph([1, 2, 31, 32, 33, 100, 129, 600, 1025, 1], 1500, 6, seed=k)
    dg = mg.to_device(g)
    rng = np.random.default_rng(k)
    kw = {"mode": mode, "k": k}
    for groups in (5, 400, g.n):
        C = rng.integers(0, groups, size=g.n).astype(np.int32)
        tC = torch.from_numpy(C).to("cuda")
        for algo, oalgo in ((mg.ALGO_LPA, oracle.ALGO_LPA), (mg.ALGO_LOUVAIN, oracle.ALGO_MOVE)):
            Cn, gain, _ = mg.move_sweep(dg, algo, tC, 0, chunk_len=L, **kw)
            eC, eg = oracle.move_sweep(g, oalgo, C, chunk_len=LONG, direction=0, **kw)
            assert np.array_equal(Cn.cpu().numpy(), eC), (groups, algo)
        D = np.unique(C, return_inverse=True)[1].astype(np.int32)
        m = int(D.max()) + 1
        for symmetric in (False, True):
            got = mg.aggregate(dg, torch.from_numpy(D).to("cuda"), m, symmetric, chunk_len=L, **kw)
            want = oracle.aggregate(g, D, m, symmetric=symmetric, chunk_len=LONG, **kw)
            for a, b in zip(got, (want.offsets, want.indices, want.weights)):
                assert np.array_equal(a, b), (groups, symmetric)


@pytest.mark.parametrize("L", [LONG + 1, (1 << 63) - 1])
@pytest.mark.parametrize("algo", ["lpa", "louvain", "leiden"])
def test_long_chunks_whole_calls(mg, algo, L):  # noqa: F811
    g = hub_graph([40, 200, 300, 1], 400, 5, seed=9)
    dg = mg.to_device(g)
    want, est = getattr(oracle, algo)(g, k=8, chunk_len=LONG)
    got, st = getattr(mg, algo)(dg, k=8, chunk_len=L)
    assert np.array_equal(got.cpu().numpy(), want) and st["iterations"] == est.iterations
    if algo != "leiden":
        labs, _, _ = mg.run_batched(mg.ALGO_LPA if algo == "lpa" else mg.ALGO_LOUVAIN, [dg, dg], k=8, chunk_len=L)
        assert all(np.array_equal(x.cpu().numpy(), want) for x in labs)
    A = {"lpa": mg.ALGO_LPA, "louvain": mg.ALGO_LOUVAIN, "leiden": mg.ALGO_LEIDEN}[algo]
    for stepped in (False, True):
        with mg.Server(A, 1 << 28, slots=2, stepped=stepped, k=8, chunk_len=L) as srv:
            lab, _, _ = srv.wait(srv.submit(dg))
            assert np.array_equal(lab.cpu().numpy(), want)
