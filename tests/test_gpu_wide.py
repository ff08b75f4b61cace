"""Several waves per cell (lanes 128) over the numbers of waves that the box
selects (4, 8, 16) and both block sizes: members on both sides of the
counting rank's bound and of a thread's particles, and acceptance rates at
which a cell's pairs take one round, several rounds, or fill a wave's list;
fused steps against one oracle step, and the collide-only last step."""
import numpy as np
import pytest

from test_gpu_parity import _cells_box, lib  # noqa: F401
from test_gpu_small_cells import _fused_step_check

pytestmark = pytest.mark.gpu

WIDE = 128
# (cells per axis, occupancies): few members (4 waves), a mean of 80-300 (8),
# more than 300 (16)
BOXES = {"4 waves": (3, [0, 1, 2, 3, 63, 64, 65, 128, 129, 255, 256, 257, 300] + [9] * 14),
         "8 waves": (2, [255, 256, 257, 190, 511, 2, 0, 130]),
         "16 waves": (2, [511, 512, 400, 700, 1, 0, 300, 257])}


@pytest.mark.parametrize("two_k", (1.0, 0.3, 0.05, 0.002))
@pytest.mark.parametrize("box", list(BOXES))
@pytest.mark.parametrize("cap", (512, 1024))
def test_wide_cells_parity(orc, lib, box, cap, two_k):  # noqa: F811
    m, occ = BOXES[box]
    V = 1.0 / m ** 3
    params = dict(box=(1.0, 1.0, 1.0), cells=(m, m, m), sigma=two_k * 0.5 * V / 0.001,
                  r_test=1.0, dt=0.001, seed=41, cell_capacity=cap)
    _fused_step_check(orc, lib, params, _cells_box(occ, m=m, seed=6), 2, WIDE,
                      f"{box} cap={cap} 2K={two_k}")


def test_wide_cells_of_one_wave_results(lib):  # noqa: F811
    from paper_1208_0961_amd import cuba as C
    m, occ = BOXES["8 waves"]
    params = dict(box=(1.0, 1.0, 1.0), cells=(m, m, m), sigma=4.0, r_test=1.0, dt=0.001,
                  seed=4, cell_capacity=512)
    out = []
    for lanes in (0, WIDE):
        s = lib.Sim(params, _cells_box(occ, m=m, seed=2), cell_lanes=lanes)
        s.step(9)
        s.step(1)
        out.append((s.get_state(), C.cuba_counters(s.ctx)))
        s.close()
    for a, b in zip(out[0][0], out[1][0]):
        assert np.array_equal(a, b)
    assert out[0][1] == out[1][1] and out[0][1]["claims"] > 0
