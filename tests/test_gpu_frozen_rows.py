"""Batches in which some graphs stop early: their rows stay where they are while the rows
beside them, in the same waves too, move on.  Against the CPU oracle, and a sweep over
rows that stay is a small part of one that moves them.  Run on an MI355X only."""
import numpy as np
import pytest

import oracle
from paper_2411_02268_amd import synth
from test_gpu_rows import hub_graph, mg  # noqa: F401 (the library's fixture)

pytestmark = pytest.mark.gpu


def cliques(count, size):
    a, b = np.triu_indices(size, 1)
    base = (np.arange(count) * size)[:, None]
    return synth.csr_from_undirected(count * size, (base + a).ravel(), (base + b).ravel(), seed=1, wmax=1)


def chain(n):
    return synth.csr_from_undirected(n, np.arange(n - 1), np.arange(1, n), seed=1, wmax=8)


@pytest.fixture(scope="module")
def graphs():
    """Cliques that stop after a sweep or two between graphs that go on; all row classes,
    sizes that are no multiple of a wave, enough short rows for 64 of them to a wave."""
    out = []
    for s in range(30):
        out.append(cliques(350 - 7 * s, 9 + s % 24))
        out.append(chain(1000 + 37 * s))
        out.append(synth.planted_exact(n_comm=4 + s % 3, comm_size=150 + s, half_intra=4, seed=s)[0])
    out.append(hub_graph([40, 200, 300, 5000], 6000, 5, seed=9))
    assert sum(int(((d := np.diff(g.offsets)) >= 8)[d <= 32].sum()) for g in out) > 2048 * 64
    return out


@pytest.mark.parametrize("kw", [{"mode": 0, "k": 8}, {"mode": 5, "k": 37}, {"mode": 1, "k": 8},
                                {"mode": 1, "k": 16, "short_rows": 2}, {"mode": 1, "k": 64}])
@pytest.mark.parametrize("algo", ["lpa", "louvain"])
def test_graphs_that_stop(mg, graphs, algo, kw):  # noqa: F811
    A = mg.ALGO_LPA if algo == "lpa" else mg.ALGO_LOUVAIN
    labs, per, _ = mg.run_batched(A, [mg.to_device(g) for g in graphs], tolerance=0.001, **kw)
    okw = {k: v for k, v in kw.items() if k != "short_rows"}
    sweeps = set()
    for i, g in enumerate(graphs):
        elab, est = getattr(oracle, algo)(g, tolerance=0.001, **okw)
        assert np.array_equal(labs[i].cpu().numpy(), elab), i
        assert per[i]["iterations"] == est.iterations, i
        sweeps.add(est.iterations)
    assert len(sweeps) > 1


def test_time_of_rows_that_stay(mg):  # noqa: F811
    """63 graphs of cliques that stop after two sweeps beside one that takes 200: 2.5 M rows
    of 23 entries that only copy their label.  That is less than a tenth of the bytes of a
    sweep that moves them."""
    gs = [mg.to_device(cliques(1666, 24)) for _ in range(63)] + [mg.to_device(chain(40000))]
    ms = {}
    for it in (1, 20, 200):
        runs = []
        for _ in range(6):
            _, per, tot = mg.run_batched(mg.ALGO_LOUVAIN, gs, mode=0, max_passes=1, tolerance=0.0, max_iterations=it)
            runs.append(tot["ms_local_move"])
        ms[it] = min(runs)
    assert per[0]["iterations"] <= 3 and per[-1]["iterations"] == 200
    stay = (ms[200] - ms[20]) / 180
    print(f"first sweep {1e3 * ms[1]:.1f} us, a sweep of rows that stay {1e3 * stay:.1f} us")
    assert stay < ms[1] / 10
