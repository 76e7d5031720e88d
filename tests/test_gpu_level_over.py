"""The rest of a step once no resident graph moves: its kernels return at once, for every
class of rows, so a long step costs its launches.  Run on an MI355X only."""
import numpy as np
import pytest

from test_gpu_frozen_rows import cliques
from test_gpu_rows import mg  # noqa: F401 (the library's fixture)

pytestmark = pytest.mark.gpu

SWEEPS = 1000


def step_ms(mg, g, **kw):  # noqa: F811
    """Least time of a step of 1000 sweeps over one graph that stops after a few."""
    dg = mg.to_device(g)
    times, labs = [], None
    with mg.Server(mg.ALGO_LPA, 4 << 30, slots=1, stepped=True, max_iterations=SWEEPS, **kw) as srv:
        for _ in range(4):
            s0 = srv.step_stats()
            labs, st, _ = srv.wait(srv.submit(dg))
            s1 = srv.step_stats()
            assert s1["sweeps"] - s0["sweeps"] == SWEEPS and st["iterations"] < 10
            times.append(s1["s_sweep"] - s0["s_sweep"])
    return 1e3 * min(times), labs.cpu().numpy()


def test_rest_of_a_step(mg):  # noqa: F811
    """2.5 M rows of 7 entries on the short rows' kernel, on the light rows', and half as many
    entries again on the main kernel.  The light rows' launch has twice the short rows'
    workgroups, which only end; with the rows gone over it takes six times as long."""
    small = cliques(2500000 // 8, 8)
    short, a = step_ms(mg, small, k=8, short_rows=2)
    light, b = step_ms(mg, small, k=8, short_rows=1)
    heavy, c = step_ms(mg, cliques(400000 // 40, 40), k=8)
    print(f"a step of {SWEEPS} sweeps: short rows {short:.2f} ms, light rows {light:.2f}, heavy rows {heavy:.2f}")
    assert np.array_equal(a, np.arange(a.size) // 8) and np.array_equal(a, b) and np.array_equal(c, np.arange(c.size) // 40)
    assert light < 3 * short and heavy < 1.5 * short
