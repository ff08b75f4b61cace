"""cuba_get_state on both sides of the size from which it exports in two
launches, with ragged and overflowing cells: every particle under its id."""
import numpy as np
import pytest

from paper_1208_0961_amd import workload as W
from test_gpu_parity import lib  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", (1, 131071, 131072, 131073, 300001))
@pytest.mark.parametrize("cells,cap", [((30, 5, 7), 0), ((64, 40, 40), 0), ((16, 4, 4), 64)])
def test_state_comes_back_by_id(lib, n, cells, cap):  # noqa: F811
    box = (10.0, 2.0, 2.0)
    state = W.thermal_box(box, n, 0.4, seed=n)
    params = dict(box=box, cells=cells, sigma=0.0, r_test=100.0, dt=0.01, seed=5,
                  cell_capacity=cap)
    sim = lib.Sim(params, state)
    got = sim.get_state()
    for a, b in zip(got, state):
        assert np.array_equal(a, b)
    sim.step(3)                 # the other buffer, whose ids the export may use
    first = sim.get_state()
    again = sim.get_state()
    sim.step(2)
    sim.close()
    whole = lib.Sim(params, state)
    whole.step(3)
    ref = whole.get_state()
    whole.close()
    for a, b, c in zip(first, again, ref):
        assert np.array_equal(a, b) and np.array_equal(a, c)
