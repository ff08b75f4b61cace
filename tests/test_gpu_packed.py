"""The packed kernel over its tile sizes (8 to 64 cells a workgroup, by the
mean occupancy and the number of cells), with units that end exactly at 64
particles and with larger cells stepped by the kernel itself (few of them)
or by a launch of their own, in LDS or in global memory; on the plain path
fused steps against one oracle step, in a batch against the lone run."""
import numpy as np
import pytest

from test_gpu_parity import lib  # noqa: F401
from test_gpu_small_cells import _fused_step_check, _grid_state

pytestmark = pytest.mark.gpu


def _occupancy(pattern, cells, mean, seed=3):
    rng = np.random.default_rng(seed)
    occ = rng.poisson(mean, cells).clip(0, 64)
    if pattern == "full units":          # units of exactly 64 and one more
        occ = np.resize([32, 32, 64, 63, 1, 1, 0, 16, 48], cells)
    if pattern == "few large":           # at most one cell in 64
        occ[[0, 200, cells - 1]] = (65, 300, 130)
    if pattern == "past the LDS":
        occ[[63, 300]] = (600, 90)
    if pattern == "many large":
        occ[::16] = 70
    return occ


@pytest.mark.parametrize("pattern", ("poisson", "full units", "few large", "past the LDS",
                                     "many large"))
@pytest.mark.parametrize("m,mean", ((8, 1.0), (8, 4.0), (8, 12.0), (9, 2.0)))
def test_packed_fused_parity(orc, lib, pattern, m, mean):  # noqa: F811
    occ = _occupancy(pattern, m ** 3, mean)
    params = dict(box=(1.0, 1.0, 1.0), cells=(m, m, m), sigma=0.02, r_test=1.0, dt=0.002,
                  seed=77, cell_capacity=128)
    _fused_step_check(orc, lib, params, _grid_state(occ, m=m, seed=m), 2, 1, f"{pattern} {m}")


@pytest.mark.parametrize("pattern", ("poisson", "few large", "past the LDS", "many large"))
@pytest.mark.parametrize("lanes,cap", ((8, 96), (32, 256), (16, 600)))
def test_packed_batch_equals_lone_run(lib, pattern, lanes, cap):  # noqa: F811
    from paper_1208_0961_amd import batch
    m = 8
    events = [(mean, dict(box=(1.0, 1.0, 1.0), cells=(m, m, m), sigma=0.02, r_test=1.0,
                          dt=0.002, seed=5 + i, cell_capacity=cap))
              for i, mean in enumerate((1.0, 6.0, 20.0))]
    states = [_grid_state(_occupancy(pattern, m ** 3, mean, seed=i), m=m, seed=i)
              for i, (mean, _) in enumerate(events)]
    B = batch.Batch(len(events))
    for i, ((_, params), st) in enumerate(zip(events, states)):
        B.admit(i, params, st)
        B.set_cell_lanes(i, lanes)
    B.step(4)
    B.sync()
    for i, ((_, params), st) in enumerate(zip(events, states)):
        s = lib.Sim(params, st, cell_lanes=0)
        s.step(4)
        ref = s.get_state()
        s.close()
        for a, b in zip(B.get_state(i), ref):
            assert np.array_equal(a, b), (pattern, i)
    B.close()
