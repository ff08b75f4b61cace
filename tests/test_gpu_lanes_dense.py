"""Lanes per cell set for boxes on both sides of the mean from which they take
a wave per cell: the states and counters of a wave per cell, and a trace of
the oracle's decisions."""
import numpy as np
import pytest

from test_gpu_parity import compare_step, lib  # noqa: F401
from test_gpu_small_cells import _grid_state

pytestmark = pytest.mark.gpu

M = 8


@pytest.mark.parametrize("mean", (29, 30, 31, 55))
def test_set_lanes_at_dense_means(orc, lib, mean):  # noqa: F811
    from paper_1208_0961_amd import cuba as C
    rng = np.random.default_rng(mean)
    occ = np.full(M ** 3, mean)
    move = rng.integers(0, mean, M ** 3 // 2)
    occ[::2] += move
    occ[1::2] -= move
    params = dict(box=(1.0, 1.0, 1.0), cells=(M, M, M), sigma=0.002, r_test=1.0, dt=0.01,
                  seed=12, cell_capacity=96)
    state = _grid_state(occ, m=M)
    ref = None
    for lanes in (0, 8, 16, 32, 64):
        s = lib.Sim(params, state, cell_lanes=lanes)
        assert s.cell_lanes == lanes
        s.step(3)
        s.step(1)
        got = (s.get_state(), C.cuba_counters(s.ctx))
        s.close()
        if ref is None:
            ref = got
            assert got[1]["claims"] > 500
        for a, b in zip(got[0], ref[0]):
            assert np.array_equal(a, b), lanes
        assert got[1] == ref[1], lanes
    for lanes in (8, 64):
        compare_step(orc, lib, params, state, 0, f"mean {mean}", lanes=lanes)
