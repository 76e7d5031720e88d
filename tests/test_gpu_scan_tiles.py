"""Vertex counts that put the scans on both sides of their tiles of 2048 items and of the one
launch that small scans take (eight tiles).  Run on an MI355X only."""
import numpy as np
import pytest

import oracle
from paper_2411_02268_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2047, 2048, 2049, 4096, 6145, 14336, 16383, 16384, 16385, 18432, 20481])
@pytest.mark.parametrize("mode", [0, 1])
def test_scans_of_few_tiles(n, mode):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_02268_amd as mg
    rng = np.random.default_rng(n)
    u, v = rng.integers(0, n, size=3 * n), rng.integers(0, n, size=3 * n)
    keep = u != v
    pairs = np.unique(np.stack([np.minimum(u, v)[keep], np.maximum(u, v)[keep]]), axis=1)
    g = synth.csr_from_undirected(n, pairs[0], pairs[1], 1 + (pairs[0] % 5).astype(np.uint32))
    dg = mg.to_device(g)
    for m in (n, n - 1, n // 3):
        D = rng.permutation(np.concatenate([np.arange(m), rng.integers(0, m, size=n - m)])).astype(np.int32)
        for symmetric in (False, True):
            off, idx, w = mg.aggregate(dg, torch.from_numpy(D).to("cuda"), m, symmetric, mode=mode, k=8)
            want = oracle.aggregate(g, D, m, mode=mode, k=8, symmetric=symmetric)
            assert np.array_equal(off, want.offsets) and np.array_equal(idx, want.indices)
            assert np.array_equal(w, want.weights)
    lab, _ = mg.louvain(dg, mode=mode)
    assert np.array_equal(lab.cpu().numpy(), oracle.louvain(g, mode=mode)[0])
