"""Calls whose kernels have more threads than one launch takes (2^32): a slot per thread
in the rows of an aggregation, a workgroup per split row.  The expected rows are the
input's own (every community one vertex, no more keys than slots).  Run on an MI355X
only."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mg():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_02268_amd as m
    m.lib()
    yield m
    torch.cuda.empty_cache()


def csr(mg, n, u, v):
    """Symmetric CSR of distinct undirected edges on the GPU, columns ascending, weights 1 .. 5."""
    import torch
    pair = torch.unique(torch.minimum(u, v) * n + torch.maximum(u, v))
    lo, hi = pair // n, pair % n
    keep = lo != hi
    lo, hi = lo[keep], hi[keep]
    w = (lo * 7 + hi * 13) % 5 + 1
    key, order = torch.sort(torch.cat([lo * n + hi, hi * n + lo]))
    off = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    off[1:] = torch.cumsum(torch.bincount(key // n, minlength=n), 0)
    return mg.DeviceGraph(off, (key % n).to(torch.int32), torch.cat([w, w])[order].to(torch.int32))


@pytest.mark.parametrize("symmetric", [False, True])
@pytest.mark.parametrize("n,k", [(1 << 24, 256), ((1 << 28) + 1000, 16)])
def test_slots(mg, symmetric, n, k):
    """2^24 communities of 256 slots and 2^28 of 16: nearly all without entries, so that no
    other kernel of the call has as many threads; the last rows are beyond the first launch."""
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    u = torch.randint(0, n, (4000,), generator=gen, device="cuda")
    v = torch.randint(0, n, (4000,), generator=gen, device="cuda")
    tail = torch.arange(n - 200, n, device="cuda")
    g = csr(mg, n, torch.cat([u, tail]), torch.cat([v, tail.flip(0)]))
    D = torch.arange(n, dtype=torch.int32, device="cuda")
    off, idx, w = mg.aggregate(g, D, n, symmetric, mode=1, k=k)
    assert (off == g.offsets.cpu().numpy()).all()
    assert (idx == g.indices.cpu().numpy()).all()
    assert (w == g.weights.cpu().numpy()).all()


def ring(mg, n, hub):
    """Two entries a row, but the last vertex has `hub` more."""
    import torch
    a = torch.arange(n, device="cuda")
    return csr(mg, n, torch.cat([a, torch.full((hub,), n - 1, device="cuda")]),
               torch.cat([(a + 1) % n, torch.arange(hub, device="cuda") * 1009 + 5]))


def test_split_streams(mg):
    """2^23 streams of 128 slots, one of two chunks: the merge tree has a workgroup each."""
    import torch
    n = (1 << 23) + 1000
    g = ring(mg, n, 100)
    D = torch.arange(n, dtype=torch.int32, device="cuda")
    off, idx, w = mg.aggregate(g, D, n, mode=1, k=128, chunk_len=64)
    assert (off == g.offsets.cpu().numpy()).all()
    assert (idx == g.indices.cpu().numpy()).all()
    assert (w == g.weights.cpu().numpy()).all()


def test_split_rows(mg):
    """2^23 split rows of a sweep, two chunks each (the unconditional rule splits every row
    at 128 slots), against 64 slots, which keep such rows in one wave and hold as much."""
    import torch
    n = (1 << 23) + 1000
    g = ring(mg, n, 0)
    C = torch.arange(n, dtype=torch.int32, device="cuda")
    for algo in (mg.ALGO_LPA, mg.ALGO_LOUVAIN):
        got, gain, ctr = mg.move_sweep(g, algo, C, 0, mode=2, k=128, chunk_len=1)
        want, wgain, wctr = mg.move_sweep(g, algo, C, 0, mode=2, k=64, chunk_len=1)
        assert wctr[0] == n and ctr == wctr
        assert torch.equal(got, want) and torch.equal(gain, wgain)


@pytest.mark.parametrize("n,k", [((1 << 26) + 1000, 64), ((1 << 24) + 1000, 128)])
def test_wave_and_workgroup_per_stream(mg, n, k):
    """A wave per stream at 64 slots; at 128 a workgroup per stream lists its chunks."""
    import torch
    g = ring(mg, n, 0)
    D = torch.arange(n, dtype=torch.int32, device="cuda")
    off, idx, w = mg.aggregate(g, D, n, mode=1, k=k)
    assert (off == g.offsets.cpu().numpy()).all()
    assert (idx == g.indices.cpu().numpy()).all()
    assert (w == g.weights.cpu().numpy()).all()


TABLES = {"mode": 0, "exact_small": 1, "exact_lds": 1}  # rows of two entries to the exact mode's tables


@pytest.mark.parametrize("n,kw,other", [
    ((1 << 26) + 1000, {"mode": 2, "k": 64}, {"mode": 2, "k": 16}),              # a wave per row
    ((1 << 26) + 1000, {**TABLES, "exact_lds": 2}, {"mode": 0}),                 # a wave per row
    ((1 << 24) + 1000, {**TABLES, "exact_lds_big": 2}, {"mode": 0}),             # a workgroup per row
    ((1 << 24) + 1000, {**TABLES, "exact_lds_big": 1}, {"mode": 0}),             # global tables
    ((1 << 24) + 1000, {"mode": 1, "k": 8, "chunk_len": 1, "row_lanes": 1}, {"mode": 0}),  # long rows
])
def test_wave_and_workgroup_per_row(mg, n, kw, other):
    """Schedules that give each of these many rows a wave or a workgroup, against one that
    does not; rows of two entries are exact in every mode."""
    import torch
    g = ring(mg, n, 0)
    C = torch.arange(n, dtype=torch.int32, device="cuda")
    for algo in (mg.ALGO_LPA, mg.ALGO_LOUVAIN):
        got, gain, ctr = mg.move_sweep(g, algo, C, 0, **kw)
        want, wgain, wctr = mg.move_sweep(g, algo, C, 0, **other)
        assert wctr[0] == n and ctr == wctr
        assert torch.equal(got, want) and torch.equal(gain, wgain)
