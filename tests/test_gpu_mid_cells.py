"""Cells that outgrow the LDS of 512 slots in boxes whose kernels have that
LDS: 513 to 1024 members in the block or past it, and more; in the one-wave,
group and packed kernels, fused and collide-only, against one oracle step, and
in a batch against the lone run."""
import numpy as np
import pytest

from test_gpu_parity import compare_step, lib  # noqa: F401
from test_gpu_small_cells import _fused_step_check, _grid_state

pytestmark = pytest.mark.gpu

SIDES = {0: (-1, 0, 0), 1: (1, 0, 0), 2: (0, -1, 0), 3: (0, 1, 0)}


def _marching(m, mean, targets, seed=3):
    """A Poisson box and, for each (cell, neighbours, n): n particles in each of
    the cell's first so many neighbours, all of which the first step (half a
    cell) carries into the cell."""
    rng = np.random.default_rng(seed)
    state = [list(a) for a in _grid_state(rng.poisson(mean, m ** 3), m=m, seed=seed)]
    for (i, j, k), sides, n in targets:
        for s in range(sides):
            d = np.array(SIDES[s])
            r = 0.1 + 0.8 * rng.random((n, 3))
            axis = int(np.argmax(np.abs(d)))
            # within 0.05 .. 0.4 of the face to the target
            off = 0.05 + 0.35 * rng.random(n)
            r[:, axis] = np.where(d[axis] > 0, off, 1.0 - off)
            r = (np.array([i, j, k]) + d + r) / m
            p = np.tile(-d * 0.6, (n, 1)) + rng.normal(size=(n, 3)) * 0.01
            for a, v in zip(state, (*r.T, *p.T)):
                a.extend(v)
    state = [np.asarray(a) for a in state]
    perm = rng.permutation(len(state[0]))
    return [np.ascontiguousarray(a[perm]) for a in state]


def _params(m, mean, cap, k=9.0):
    return dict(box=(1.0, 1.0, 1.0), cells=(m, m, m), r_test=1.0, dt=0.5 / m,
                sigma=k / mean ** 2 / m ** 3 / (0.5 / m), seed=19, cell_capacity=cap)


def _counts(state, m):
    i = [np.minimum((a * m).astype(np.int64), m - 1) for a in state[:3]]
    return np.bincount((i[0] * m + i[1]) * m + i[2], minlength=m ** 3)


# members: 2 x 240 + some of the box (below 513 or not), 2 x 320, 3 x 320, 4 x 320
TARGETS = [((1, 1, 1), 2, 240), ((3, 2, 2), 2, 320), ((5, 5, 5), 3, 320), ((2, 6, 4), 4, 320),
           ((6, 6, 1), 2, 256)]


@pytest.mark.parametrize("nsteps", (1, 2))
@pytest.mark.parametrize("m,mean,lanes", [(8, 40, 0), (19, 54, 0), (8, 40, 16), (8, 40, 128)])
@pytest.mark.parametrize("cap", (1024, 640, 512, 96))
def test_outgrown_cells(orc, lib, m, mean, lanes, cap, nsteps):  # noqa: F811
    state = _marching(m, mean, TARGETS)
    params = _params(m, mean, cap)
    before = _counts(state, m)
    assert before.max() <= 384 and (m < 19 or before.mean() >= 50)
    s = lib.Sim(params, state, cell_lanes=lanes)
    s.step(1)
    after = np.sort(_counts(s.get_state(), m))
    s.close()
    assert after[-1] > 1024 and np.sum((after > 512) & (after <= 1024)) >= 2
    assert _fused_step_check(orc, lib, params, state, nsteps, lanes, f"cap {cap}") > 500


@pytest.mark.parametrize("lanes", (0, 16, 128))
@pytest.mark.parametrize("cap", (1024, 512, 96))
def test_outgrown_cells_traced(orc, lib, lanes, cap):  # noqa: F811
    _, tr = compare_step(orc, lib, _params(8, 40, cap), _marching(8, 40, TARGETS), 0,
                         f"outgrown, cap {cap}", lanes=lanes)
    assert len(tr["claim"]) > 500


@pytest.mark.parametrize("lanes", (0, 16))
def test_outgrown_cells_in_a_batch(lib, lanes):  # noqa: F811
    from paper_1208_0961_amd import batch
    from paper_1208_0961_amd import cuba as C
    m, mean = 19, 54
    state = _marching(m, mean, TARGETS)
    for cap in (512, 640):
        B = batch.Batch(1)
        B.admit(0, _params(m, mean, cap), state)
        B.set_cell_lanes(0, lanes)
        obs = B.set_observe(0, 1, rows=3)
        B.step(3)
        B.sync()
        s = lib.Sim(_params(m, mean, cap), state, cell_lanes=0)
        for k in (1, 2, 3):
            s.step(1)
            T00, T0x = s.observe()
            tol = 2.0 * len(state[0]) * 2.0 ** -53
            got = obs[k % 3].cpu().numpy()
            assert np.all(np.abs(got[0] - T00) <= tol * T00)
            assert np.all(np.abs(got[1] - T0x) <= tol * T00)
        for a, b in zip(B.get_state(0), s.get_state()):
            assert np.array_equal(a, b)
        assert C.cuba_counters(B.ctx(0)) == C.cuba_counters(s.ctx)
        s.close()
        B.close()
