"""Row sums, total weight and modularity where rows and tiles of 2048 entries meet: rows that
end with a tile, cross one or several, empty rows between them, and a last tile of a few
entries.  Whole numbers, so the weights agree exactly and the quotient to rounding (a few
operations of 2^-53 each).  Run on an MI355X only."""
import numpy as np
import pytest

import oracle
from paper_2411_02268_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hubs", [[1], [1023], [1024], [1024, 1], [1025], [2047, 3, 2048], [5000, 7, 4096, 1]])
@pytest.mark.parametrize("wmax", [1, 9, 1 << 16])
def test_tile_edges(hubs, wmax):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_02268_amd as mg
    rng = np.random.default_rng(sum(hubs))
    n = 6000 + 2 * len(hubs)  # every second hub id has no entries, as most leaves
    edges, ws = [], []
    for h, deg in enumerate(hubs):
        for v in rng.choice(6000, size=deg, replace=False):
            edges.append((int(v), 6000 + 2 * h))
            ws.append(int(rng.integers(1, wmax + 1)))
    g = synth.from_edges(n, edges, weights=ws)
    dg = mg.to_device(g)
    for groups in (1, 5, n):
        C = rng.integers(0, groups, size=n).astype(np.int32)
        q = mg.modularity(dg, torch.from_numpy(C).to("cuda"))
        assert abs(q - oracle.modularity(g, C)) <= 1e-14
