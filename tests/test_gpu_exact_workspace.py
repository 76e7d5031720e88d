"""Calls in exactly the workspace they state, with a mark behind it: every array that they
take lies inside, whatever the sizes.  Run on an MI355X only."""
import ctypes as ct

import numpy as np
import pytest

import oracle
from paper_2411_02268_amd import synth
from test_gpu_rows import hub_graph, mg  # noqa: F401 (the library's fixture)

pytestmark = pytest.mark.gpu

MARK = 4096


def guarded(nbytes):
    import torch
    return torch.full((nbytes + MARK,), 0xA5, dtype=torch.uint8, device="cuda")


def intact(ws, nbytes):
    return bool((ws[nbytes:] == 0xA5).all())


GRAPHS = {
    "one": lambda: synth.from_edges(1, [], self_loops={0: 2}),
    "pairs": lambda: synth.from_edges(2000, [(2 * i, 2 * i + 1) for i in range(1000)]),
    "hubs": lambda: hub_graph([1, 40, 200, 300, 5000, 9000], 9500, 5, seed=9),
    "rmat": lambda: synth.rmat(scale=13, edge_factor=12, seed=3),
}


@pytest.mark.parametrize("graph", sorted(GRAPHS))
@pytest.mark.parametrize("mode,k,L", [(1, 1, 1), (1, 8, 128), (3, 16, 1), (1, 64, 3), (2, 128, 128), (1, 256, 1),
                                      (0, 8, 128), (5, 9, 128)])
@pytest.mark.parametrize("symmetric", [0, 1])
def test_aggregate(mg, graph, mode, k, L, symmetric):  # noqa: F811
    import torch
    g = GRAPHS[graph]()
    dg = mg.to_device(g)
    p = mg.params(mg.ALGO_LEIDEN, mode=mode, k=k, k_aggregate=k if mode != 5 else 8, chunk_len=L)
    for m in {1, (g.n + 2) // 3, g.n}:
        D = (np.arange(g.n) * 7919 % m).astype(np.int32) if m < g.n else np.arange(m, dtype=np.int32)
        D = np.unique(D, return_inverse=True)[1].astype(np.int32)
        m = int(D.max()) + 1
        tD = torch.from_numpy(D).to("cuda")
        off = torch.empty(m + 1, dtype=torch.int64, device="cuda")
        idx = torch.empty(max(g.nnz, 1), dtype=torch.int32, device="cuda")
        w = torch.empty(max(g.nnz, 1), dtype=torch.int32, device="cuda")
        nnz, d = ct.c_int64(), dg.desc()

        def call(ws, nbytes):
            return mg.lib().mgcd_aggregate(ct.byref(d), ct.byref(p), tD.data_ptr(), m, symmetric, off.data_ptr(),
                                           idx.data_ptr(), w.data_ptr(), ct.byref(nnz), ws.data_ptr(), nbytes,
                                           mg._stream())
        assert call(guarded(0), 0) == -4  # and the message states the bytes
        nbytes = int(mg.lib().mgcd_last_error().decode().split("needs ")[1].split()[0])
        ws = guarded(nbytes)
        mg._check(call(ws, nbytes))
        assert intact(ws, nbytes)
        want = oracle.aggregate(g, D, m, symmetric=bool(symmetric), mode=0 if mode == 5 else mode, k=k, chunk_len=L)
        e = nnz.value
        assert np.array_equal(off.cpu().numpy(), want.offsets) and np.array_equal(idx[:e].cpu().numpy(), want.indices)
        assert np.array_equal(w[:e].cpu().numpy().view(np.uint32), want.weights)


@pytest.mark.parametrize("graph", sorted(GRAPHS))
@pytest.mark.parametrize("algo", ["lpa", "louvain", "leiden"])
@pytest.mark.parametrize("kw", [{"k": 8}, {"k": 16, "chunk_len": 1, "storage_order": 2}, {"k": 64}, {"k": 128, "mode": 2},
                                {"mode": 0}, {"mode": 0, "exact_small": 1, "exact_lds": 1, "exact_lds_big": 1}])
def test_whole_calls(mg, graph, algo, kw):  # noqa: F811
    import torch
    g = GRAPHS[graph]()
    dg = mg.to_device(g)
    A = {"lpa": mg.ALGO_LPA, "louvain": mg.ALGO_LOUVAIN, "leiden": mg.ALGO_LEIDEN}[algo]
    p = mg.params(A, **kw)
    nbytes = int(mg.lib().mgcd_workspace_bytes(A, dg.n, dg.nnz, ct.byref(p)))
    ws = guarded(nbytes)
    out = torch.empty(g.n, dtype=torch.int32, device="cuda")
    d = dg.desc()
    mg._check(getattr(mg.lib(), algo + "_run")(ct.byref(d), ct.byref(p), out.data_ptr(), ws.data_ptr(), nbytes, None,
                                               mg._stream()))
    assert intact(ws, nbytes)
    okw = {x: v for x, v in kw.items() if x in ("k", "mode", "chunk_len")}
    assert np.array_equal(out.cpu().numpy(), getattr(oracle, algo)(g, **okw)[0])
