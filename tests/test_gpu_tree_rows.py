"""The split rows and streams of the wide sketches that take part in the merge tree: lengths
on both sides of one node and of the classes that lists are ordered by, among many rows of
one node.  Against the CPU oracle, bit for bit, and one long row does not make the others
pay for its tree.  Run on an MI355X only."""
import numpy as np
import pytest

import oracle
from test_gpu_rows import MODES, hub_graph, mg  # noqa: F401 (the library's fixture)

pytestmark = pytest.mark.gpu

CASES = [  # k, mode, chunk length, row lengths
    (128, "uncond", 31, [1, 2, 30, 31, 32, 33, 62, 63, 64, 65, 93, 94]),
    (128, "uncond", 32, [1, 31, 32, 33, 34, 63, 64, 65, 2049, 2050]),
    (128, "alg1", 33, [33, 34, 63, 64, 65, 66, 67, 127, 128, 129, 2112, 2113]),
    (256, "alg1", 40, [33, 40, 41, 80, 81, 2560, 2561, 2600]),
    (256, "uncond", 1, [1, 2, 3, 31, 32, 33, 64, 65, 130]),
    (64, "alg1", 64, [511, 512, 513, 514, 1023, 1024, 1025, 2048, 2049]),
    (64, "std", 63, [504, 505, 513, 1008, 1009, 4032, 4033]),
    (32, "uncond", 3, [511, 512, 513, 1536, 1537, 1560]),
    (32, "alg1", 100, [513, 799, 800, 801, 1023, 1024, 1600, 1601]),
]


@pytest.mark.parametrize("k,mode,L,lens", CASES)
@pytest.mark.parametrize("order", [1, -1])
def test_tree_rows(mg, k, mode, L, lens, order):  # noqa: F811
    import torch
    g = hub_graph((lens * 3)[::order], 4100, 6, seed=k + L)
    dg = mg.to_device(g)
    rng = np.random.default_rng(k)
    kw = {"mode": MODES[mode], "k": k, "chunk_len": L}
    for groups in (3, k + 20, g.n):
        C = rng.integers(0, groups, size=g.n).astype(np.int32)
        tC = torch.from_numpy(C).to("cuda")
        for algo, oalgo in ((mg.ALGO_LPA, oracle.ALGO_LPA), (mg.ALGO_LOUVAIN, oracle.ALGO_MOVE)):
            Cn, gain, _ = mg.move_sweep(dg, algo, tC, 0, **kw)
            eC, eg = oracle.move_sweep(g, oalgo, C, direction=0, **kw)
            assert np.array_equal(Cn.cpu().numpy(), eC), (groups, algo)
        D = np.arange(g.n, dtype=np.int32) if groups == g.n else (np.arange(g.n) % groups).astype(np.int32)
        m = int(D.max()) + 1
        for symmetric in (False, True):
            got = mg.aggregate(dg, torch.from_numpy(D).to("cuda"), m, symmetric, **kw)
            want = oracle.aggregate(g, D, m, symmetric=symmetric, **kw)
            for a, b in zip(got, (want.offsets, want.indices, want.weights)):
                assert np.array_equal(a, b), (groups, symmetric)


def test_time_of_one_long_row(mg):  # noqa: F811
    """A sweep over 2^21 rows of two entries, all split (the unconditional rule at 256 slots),
    with and without one row of 100,000 more: 782 nodes and their ten levels of merges, some
    tens of microseconds, where a fifth of the sweep is allowed."""
    import torch
    n = 1 << 21
    ms = []
    for hub in (0, 100000):
        a = torch.arange(n, device="cuda")
        u = torch.cat([a, torch.full((hub,), n - 1, device="cuda")])
        v = torch.cat([(a + 1) % n, torch.arange(hub, device="cuda") * 7 + 3])
        src = torch.cat([u, v])
        dst = torch.cat([v, u])
        key, _ = torch.sort(src * n + dst)
        off = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
        off[1:] = torch.cumsum(torch.bincount(key // n, minlength=n), 0)
        g = mg.DeviceGraph(off, (key % n).to(torch.int32), torch.ones(key.numel(), dtype=torch.int32, device="cuda"))
        t = []
        for _ in range(4):
            _, st = mg.lpa(g, mode=2, k=256, max_iterations=8, tolerance=0.0)
            t.append(st["ms_local_move"] / st["iterations"])
        ms.append(min(t))
    print(f"a sweep without the long row {ms[0]:.3f} ms, with it {ms[1]:.3f} ms")
    assert ms[1] < 1.2 * ms[0]
