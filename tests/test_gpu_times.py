"""The call's own times: level-0 classes that have rows get a positive device time, empty
ones none, and the parts lie within the whole (events and the device clock tick apart by
less than a percent).  Run on an MI355X only."""
import pytest

from paper_2411_02268_amd import synth

pytestmark = pytest.mark.gpu

CASES = [  # graph, parameters, classes with rows at level 0
    (lambda: synth.planted_exact(n_comm=8, comm_size=60, seed=5)[0], {"k": 8}, [True, False, False]),
    (lambda: synth.kmer_like(3000, seed=7), {"k": 8, "short_rows": 2}, None),
    (lambda: synth.rmat(scale=11, edge_factor=8, seed=3), {"k": 8, "chunk_len": 2}, [True, True, False]),
    (lambda: synth.rmat(scale=11, edge_factor=8, seed=3), {"k": 64}, None),
    (lambda: synth.rmat(scale=11, edge_factor=8, seed=3), {"mode": 0}, None),
]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("algo", ["lpa", "louvain", "leiden"])
def test_class_times(algo, case):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_02268_amd as mg
    make, kw, classes = CASES[case]
    dg = mg.to_device(make())
    for _ in range(2):
        _, st = getattr(mg, algo)(dg, **kw)
        ms = st["ms_l0_kernel"]
        assert 1 <= st["l0_sweeps"] <= st["iterations"]
        assert max(ms) > 0 and min(ms) >= 0
        if classes:
            assert [m > 0 for m in ms] == classes
        assert sum(ms) <= 1.01 * st["ms_local_move"]
        assert st["ms_local_move"] + st["ms_refine"] + st["ms_aggregate"] <= 1.01 * st["ms_total"]
        assert (st["ms_refine"] > 0) == (algo == "leiden")
