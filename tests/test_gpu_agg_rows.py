"""Aggregation streams at the edges of its kernel: 1 to 64 chunks in every bucket, aligned
groups of 64 chunks and a last group of one, chunks that end within a lane's quarter of 16
positions.  Against the CPU oracle, bit for bit.  Run on an
MI355X only."""
import numpy as np
import pytest

import oracle
from test_gpu_rows import MODES, hub_graph, mg  # noqa: F401 (the library's fixture)

pytestmark = pytest.mark.gpu

EDGES = {  # chunk length -> stream lengths
    1: [1, 2, 3, 4, 5, 8, 9, 16, 17, 32, 33, 63, 64, 65, 128, 129],
    20: [1, 19, 20, 21, 40, 41, 81, 161, 321, 641, 1279, 1280, 1281, 1300, 2561],
    128: [3, 15, 16, 17, 31, 33, 63, 64, 65, 127, 128, 129, 255, 257, 513, 1025, 2049, 4097, 8192, 8193],
}


@pytest.mark.parametrize("mode", ["alg1", "uncond", "std"])
@pytest.mark.parametrize("k", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("L", sorted(EDGES))
@pytest.mark.parametrize("symmetric", [False, True])
def test_agg_rows(mg, mode, k, L, symmetric):  # noqa: F811
    import torch
    lens = EDGES[L]
    g = hub_graph(lens, 8400, 6, seed=k + L)
    dg = mg.to_device(g)
    for groups in (3, k, 2 * k + 1, 700):
        D = (np.arange(g.n) * 7919 % groups).astype(np.int32)
        D[-len(lens):] = groups + np.arange(len(lens))  # each hub alone
        m = int(D.max()) + 1
        got = mg.aggregate(dg, torch.from_numpy(D).to("cuda"), m, symmetric, mode=MODES[mode], k=k, chunk_len=L)
        want = oracle.aggregate(g, D, m, mode=MODES[mode], k=k, chunk_len=L, symmetric=symmetric)
        for a, b in zip(got, (want.offsets, want.indices, want.weights)):
            assert np.array_equal(a, b), groups
