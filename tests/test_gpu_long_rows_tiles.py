"""Rows of many tiles of 2,048 entries: their sums and the modularity of a membership,
against integers known in advance, in no more time than short rows take.  Run on an
MI355X only."""
import numpy as np
import pytest

import oracle
from paper_2411_02268_amd import synth
from test_gpu_rows import mg  # noqa: F401 (the library's fixture)

pytestmark = pytest.mark.gpu


def rows_graph(mg, lens, n):  # noqa: F811
    """Rows of the given lengths, entry e of row i pointing at vertex (i + e) mod n, weight 1."""
    import torch
    off = torch.zeros(len(lens) + 1, dtype=torch.int64, device="cuda")
    off[1:] = torch.cumsum(torch.tensor(lens, device="cuda"), 0)
    nnz = int(off[-1])
    idx = torch.empty(nnz, dtype=torch.int32, device="cuda")
    for i, (a, b) in enumerate(zip(off.tolist(), off.tolist()[1:])):
        idx[a:b] = (torch.arange(i, i + b - a, device="cuda") % n).to(torch.int32)
    return mg.DeviceGraph(off, idx, torch.ones(nnz, dtype=torch.int32, device="cuda"))


T = 2048


@pytest.mark.parametrize("lens", [[T * 8, T * 9], [T * 8 + 1, 0, T * 8 - 1, 1], [1, T * 9, 1], [T * 200 + 5] * 3,
                                  [0] * 70 + [T * 500 + 77] + [3] * 200 + [T * 10] * 100, [T * 30000 + 1, 5]])
def test_rows_of_many_tiles(mg, lens):  # noqa: F811
    """The first rows of tiles at the edges of the rule for long rows."""
    import torch
    n = len(lens)
    g = rows_graph(mg, lens, n)
    C = torch.arange(n, dtype=torch.int32, device="cuda") // 2
    q = mg.modularity(g, C)
    inside, tot = 0, np.zeros(n, dtype=np.int64)
    c = C.cpu().numpy()
    for i, d in enumerate(lens):  # entry e of row i is vertex (i + e) mod n
        count = np.full(n, d // n)
        count[(i + np.arange(d % n)) % n] += 1
        inside += int(count[c == c[i]].sum())
        tot[c[i]] += d
    W = sum(lens)
    assert q == inside / W - float((tot * tot).sum()) / (float(W) * W)


def test_time_of_long_rows(mg):  # noqa: F811
    """2^29 entries in two rows and in 2^18: the same bytes.  The two rows' sums are one add
    per tile onto one address each; marking their 2^17 tiles (in two tables) one by one, at
    26 ns each, would be 6.8 ms on top, and less than half of that is allowed for both."""
    import torch
    ms = []
    for n in (2, 1 << 18):
        nnz = 1 << 29
        off = torch.arange(n + 1, dtype=torch.int64, device="cuda") * (nnz // n)
        idx = (torch.arange(nnz, device="cuda", dtype=torch.int32) // 2048 + 1) % n
        g = mg.DeviceGraph(off, idx.to(torch.int32), torch.ones(nnz, dtype=torch.int32, device="cuda"))
        C = torch.arange(n, dtype=torch.int32, device="cuda")
        t = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            mg.modularity(g, C)
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        ms.append(min(t))
    print(f"two rows {ms[0]:.3f} ms, 2^18 rows {ms[1]:.3f} ms")
    assert ms[0] - ms[1] < 3.4
