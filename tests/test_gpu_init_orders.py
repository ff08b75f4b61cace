"""Initial states in orders that carry position (sorted by cell, cells in
turn, one cell after a shuffled rest): every particle is binned once, under
its id, and the first step is the oracle's."""
import numpy as np
import pytest

from test_gpu_parity import compare_step, lib  # noqa: F401
from test_gpu_small_cells import _grid_state

pytestmark = pytest.mark.gpu


def _ordered(order, m, mean):
    rng = np.random.default_rng(m)
    occ = rng.poisson(mean, m ** 3)
    occ[-1] = 130
    state = _grid_state(occ, m=m)          # sorted by cell
    n = len(state[0])
    if order == "in turn":                 # the cells' first particles, their second ones, ...
        first = np.cumsum(occ) - occ
        perm = np.argsort(np.arange(n) - np.repeat(first, occ), kind="stable")
    elif order == "two at once":           # a wave's lanes in two cells, alternating
        perm = np.arange(n)[:n // 2 * 2].reshape(2, -1).T.ravel()
        perm = np.concatenate([perm, np.arange(n)[n // 2 * 2:]])
    elif order == "shuffled, then one cell":
        perm = np.concatenate([rng.permutation(n - 130), np.arange(n - 130, n)])
    else:
        perm = np.arange(n)
    return [np.ascontiguousarray(a[perm]) for a in state]


@pytest.mark.parametrize("order", ("sorted", "in turn", "two at once", "shuffled, then one cell"))
@pytest.mark.parametrize("m,mean,cap", [(4, 70, 0), (12, 3, 0), (12, 20, 16)])
def test_initial_order(orc, lib, order, m, mean, cap):  # noqa: F811
    state = _ordered(order, m, mean)
    params = dict(box=(1.0, 1.0, 1.0), cells=(m, m, m), sigma=0.02 / m ** 2, r_test=1.0,
                  dt=0.1 / m, seed=8, cell_capacity=cap)
    s = lib.Sim(params, state)
    for a, b in zip(s.get_state(), state):
        assert np.array_equal(a, b)
    s.close()
    compare_step(orc, lib, params, state, 0, order)
