"""Vertices without entries: at the end, in the middle and at the start, more of them than
entries.  Whole calls and modularity against the CPU oracle, and a graph followed by eight
million of them costs its own work and a pass over them.  Run on an MI355X only."""
import numpy as np
import pytest

import oracle
from paper_2411_02268_amd import synth
from test_gpu_rows import mg  # noqa: F401 (the library's fixture)

pytestmark = pytest.mark.gpu


def spread(g, before, every, after):
    """g with `before` empty rows first, one after each `every` vertices, and `after` at the end."""
    new = before + np.arange(g.n) + (np.arange(g.n) // every if every else 0)
    n = int(new[-1]) + 1 + after
    deg = np.zeros(n, dtype=np.int64)
    deg[new] = np.diff(g.offsets)
    off = np.concatenate([[0], np.cumsum(deg)])
    return synth.CSR(off, new[g.indices].astype(np.int32), g.weights)


@pytest.mark.parametrize("before,every,after", [(0, 0, 1), (0, 0, 5000), (3, 1, 2), (4000, 7, 0), (0, 300, 70000)])
@pytest.mark.parametrize("edge_factor", [1, 8])
def test_empty_rows(mg, before, every, after, edge_factor):  # noqa: F811
    g = spread(synth.rmat(scale=11, edge_factor=edge_factor, seed=5), before, every, after)
    dg = mg.to_device(g)
    for algo in ("lpa", "louvain", "leiden"):
        for kw in ({"mode": 1, "k": 8}, {"mode": 0}):
            lab, _ = getattr(mg, algo)(dg, **kw)
            want, _ = getattr(oracle, algo)(g, **kw)
            assert np.array_equal(lab.cpu().numpy(), want), (algo, kw)
        q, eq = mg.modularity(dg, lab), oracle.modularity(g, want)
        assert abs(q - eq) <= 1e-12
        assert mg.modularity_noalloc(dg, lab) == q


def test_time_of_empty_rows_at_the_end(mg):  # noqa: F811
    """Modularity of 2^18 entries alone and with 2^23 vertices without any behind them: those
    need their labels checked, sums zeroed and squared, some 200 MB in all, 0.1 ms at 2 TB/s."""
    import torch
    base = synth.rmat(scale=14, edge_factor=8, seed=5)
    ms = []
    for after in (0, 1 << 23):
        g = mg.to_device(spread(base, 0, 0, after))
        C = torch.arange(g.n, dtype=torch.int32, device="cuda")
        t = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            mg.modularity(g, C)
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        ms.append(min(t))
    print(f"alone {ms[0]:.3f} ms, with empty rows {ms[1]:.3f} ms")
    assert ms[1] < ms[0] + 1.0
