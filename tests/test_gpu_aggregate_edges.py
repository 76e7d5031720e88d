"""Aggregation at the edges of the sort's tiles (4,096 items, 1,024 per wave) and digits
(256 communities per pass), with diagonal entries, communities that keep no pair and
rows kept in one direction only.  Against the CPU oracle, bit for bit.  Run on an MI355X
only."""
import numpy as np
import pytest

import oracle
from paper_2411_02268_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mg():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_02268_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("n,m", [(2, 1), (2, 2), (63, 1), (1023, 255), (1024, 256), (1025, 257), (4095, 1),
                                 (4096, 4096), (4097, 65), (8193, 300), (70000, 66000)])
@pytest.mark.parametrize("mode,k", [(0, 8), (1, 2), (1, 8), (1, 16), (3, 4), (1, 64)])
@pytest.mark.parametrize("symmetric", [False, True])
def test_aggregate_edges(mg, n, m, mode, k, symmetric):
    import torch
    rng = np.random.default_rng(n + m)
    u, v = rng.integers(0, n, size=(2, 3 * n))
    # a star, so that some community has many more reversed than kept pairs, and self-loops
    u, v = np.concatenate([u, np.zeros(n // 2, np.int64)]), np.concatenate([v, np.arange(n // 2)])
    g = synth.csr_from_undirected(n, u, v, seed=n, wmax=7)
    D = np.concatenate([np.arange(m), rng.integers(0, m, size=n - m)]).astype(np.int32)
    rng.shuffle(D)
    off, idx, w = mg.aggregate(mg.to_device(g), torch.from_numpy(D).to("cuda"), m, symmetric, mode=mode, k=k)
    e = oracle.aggregate(g, D, m, symmetric=symmetric, mode=mode, k=k)
    assert np.array_equal(off, e.offsets)
    assert np.array_equal(idx, e.indices)
    assert np.array_equal(w, e.weights)
