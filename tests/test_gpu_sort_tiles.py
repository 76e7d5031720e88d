"""Graphs whose vertex and entry counts put the radix sorts on both sides of the tile order
(128 tiles of 4096 items) and leave a last tile that is nearly empty or full.  Run on an
MI355X only."""
import numpy as np
import pytest

import oracle
from paper_2411_02268_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4096 * 127, 4096 * 128 - 4095, 4096 * 128 + 1, 4096 * 131])
@pytest.mark.parametrize("mode", [0, 1])
def test_sorts_of_many_tiles(n, mode):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_02268_amd as mg
    u = np.arange(n - 1, dtype=np.int64)
    g = synth.csr_from_undirected(n, u, u + 1, 1 + (u % 5).astype(np.uint32))
    rng = np.random.default_rng(n)
    m = n // 3
    D = rng.integers(0, m, size=n).astype(np.int32)
    D[:m] = np.arange(m)
    off, idx, w = mg.aggregate(mg.to_device(g), torch.from_numpy(D).to("cuda"), m, mode=mode, k=8)
    want = oracle.aggregate(g, D, m, mode=mode, k=8)
    assert np.array_equal(off, want.offsets) and np.array_equal(idx, want.indices) and np.array_equal(w, want.weights)
