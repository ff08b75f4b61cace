"""Profiles and export of boxes in which many cells overflow their blocks,
several of them among the cells of one wave, for every number of lanes a cell:
each spilled particle counted once, in its own cell's slab, and exported under
its id."""
import numpy as np
import pytest

from test_gpu_parity import lib  # noqa: F401
from test_gpu_small_cells import _grid_state

pytestmark = pytest.mark.gpu


# (cells per axis, mean, slots): 8, 16, 32 and 64 lanes a cell
@pytest.mark.parametrize("m,mean,cap", [(48, 2, 2), (24, 12, 11), (24, 25, 20), (16, 50, 45)])
def test_spilled_particles_once_each(lib, m, mean, cap):  # noqa: F811
    rng = np.random.default_rng(m + mean)
    occ = rng.poisson(mean, m ** 3)
    occ[[0, 1, m ** 3 - 1]] = (cap + 70, cap + 1, cap + 2)
    assert np.mean(occ > cap) > 0.25 and occ.sum() >= 1 << 17
    state = _grid_state(occ, m=m)
    params = dict(box=(1.0, 1.0, 1.0), cells=(m, m, m), sigma=0.0, r_test=1.0, dt=0.3 / m,
                  seed=1, cell_capacity=cap)
    s = lib.Sim(params, state)
    for steps in (0, 1, 2):      # both buffers and both counter sets
        s.step(steps)
        T00, T0x = s.observe()
        got = s.get_state()
        if steps == 0:
            for a, b in zip(got, state):
                assert np.array_equal(a, b)
        E = np.sqrt(got[3] ** 2 + got[4] ** 2 + got[5] ** 2)
        ix = np.minimum(np.floor(got[0] / (1.0 / m)).astype(np.int64), m - 1)
        sE = np.bincount(ix, E, m) * m
        sP = np.bincount(ix, got[3], m) * m
        # two orders of a slab's sum of at most 2^17 terms
        tol = 2.0 * 2 ** 17 * 2.0 ** -53
        assert np.all(np.abs(T00 - sE) <= tol * sE)
        assert np.all(np.abs(T0x - sP) <= tol * sE)
    s.close()
