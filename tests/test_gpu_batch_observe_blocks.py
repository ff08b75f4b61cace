"""Observation inside runs of a packed event whose blocks exceed the small LDS:
its cells of more than 64 particles are stepped by a launch of their own, and
the profiles hold every cell's energy and momentum, as the lone run's do."""
import numpy as np
import pytest

from test_gpu_parity import lib  # noqa: F401
from test_gpu_small_cells import _grid_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graphs", (False, True))
@pytest.mark.parametrize("m", (16, 100))   # tiles that all run at once; many in turn
def test_profiles_hold_the_larger_cells(lib, m, graphs):  # noqa: F811
    from paper_1208_0961_amd import batch
    rng = np.random.default_rng(2)
    occ = rng.poisson(1, m ** 3)
    large = rng.choice(m ** 3, m ** 3 // 1000, replace=False)
    occ[large] = rng.integers(65, 301, len(large))
    state = _grid_state(occ, m=m)
    params = dict(box=(1.0, 1.0, 1.0), cells=(m, m, m), sigma=0.002 / m ** 2, r_test=1.0,
                  dt=0.05 / m, seed=9, cell_capacity=600)
    steps, every = 6, 2
    B = batch.Batch(2, use_graphs=graphs)
    B.admit(0, params, state)
    B.set_cell_lanes(0, 16)
    obs = B.set_observe(0, every, rows=steps // every)
    B.step(steps)
    B.sync()
    got = obs.cpu().numpy()
    B.close()
    s = lib.Sim(params, state, cell_lanes=0)
    for k in range(1, steps // every + 1):
        s.step(every)
        T00, T0x = s.observe()
        row = got[k % (steps // every)]
        # sums of the particles of a slab in two orders
        tol = 2.0 * len(state[0]) * 2.0 ** -53
        for a, b in ((row[0], T00), (row[1], T0x)):
            dev = np.abs(a - b) / T00
            assert dev.max() <= tol, (k * every, dev.max(), int((dev > tol).sum()))
    s.close()
