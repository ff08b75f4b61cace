"""The kernel in which four cells share their pairs, on boxes that are sure to
take it (the selection's rule is asserted): empty, single and few-particle
cells beside dense ones, lists of filtered pairs past their 256 entries (the
count is computed here), cells past their block; states against one oracle
step, the counters of pairs, candidates and claims against the oracle's, and a
batched event's state, counters and profiles against the lone run's."""
import numpy as np
import pytest

from test_gpu_parity import _orc_params, _rows, lib  # noqa: F401
from test_gpu_small_cells import _fused_step_check, _grid_state

pytestmark = pytest.mark.gpu

M = 19   # 6859 cells: the last group holds 3
M32 = np.uint64(0xFFFFFFFF)


def _occupancy(pattern):
    rng = np.random.default_rng(7)
    if pattern == "ragged":
        occ = rng.poisson(88, M ** 3)
        occ[::5] = rng.integers(0, 4, len(occ[::5]))
        occ[1::5] = 120
        occ[[0, 1, 2, 3, 6856, 6857, 6858]] = (0, 1, 2, 90, 0, 60, 1)
        occ[40:44] = 0
        occ[44:48] = 1
    else:
        occ = rng.poisson(72, M ** 3)
    if pattern == "lists overflow":
        occ[[3, 100, 101, 6858]] = (450, 440, 430, 450)
    if pattern == "blocks overflow":
        occ[[0, 77, 78, 6857]] = (600, 140, 300, 700)
    return occ


def _params(occ, pattern):
    """K times the mean is 0.2: some 0.2 filtered pairs a particle."""
    return dict(box=(1.0, 1.0, 1.0), cells=(M, M, M), r_test=1.0, dt=0.002,
                sigma=0.2 / float(np.mean(occ)) / M ** 3 / 0.002, seed=17,
                cell_capacity=128 if pattern == "blocks overflow" else 512)


def _takes_group_kernel(occ, params):
    """The selection's rule, alone and in a batch."""
    mean = float(np.mean(occ))
    K = params["sigma"] / params["r_test"] * params["dt"] * M ** 3
    return len(occ) >= 6000 and mean >= 66.0 and K * mean <= 0.3


def _w1(k, cell, step, key):
    """Word w1 of the Philox4x32-10 blocks of counters (k, cell, step, 0)."""
    x = [k.astype(np.uint64)] + [np.full(len(k), v, np.uint64) for v in (cell, step, 0)]
    for r in range(10):
        a, b = x[0] * np.uint64(0xD2511F53), x[2] * np.uint64(0xCD9E8D57)
        ka = np.uint64((key + r * 0x9E3779B9) & 0xFFFFFFFF)
        kb = np.uint64((r * 0xBB67AE85) & 0xFFFFFFFF)
        x = [((b >> np.uint64(32)) ^ x[1] ^ ka) & M32, b & M32,
             ((a >> np.uint64(32)) ^ x[3] ^ kb) & M32, a & M32]
    return x[1]


def _filtered(n, cell, step, params):
    """Pairs of an n-member cell that pass the w1 filter."""
    K = params["sigma"] / params["r_test"] * params["dt"] * M ** 3
    w1 = _w1(np.arange(n * (n - 1) // 2), cell, step, params["seed"])
    return int(np.sum(w1 < np.ceil(2.0 * K * 2.0 ** 32)))


PATTERNS = ("poisson", "ragged", "lists overflow", "blocks overflow")


@pytest.mark.parametrize("nsteps", (1, 2))
@pytest.mark.parametrize("pattern", PATTERNS)
def test_group_states(orc, lib, pattern, nsteps):  # noqa: F811
    occ = _occupancy(pattern)
    params = _params(occ, pattern)
    assert _takes_group_kernel(occ, params)
    state = _grid_state(occ, m=M)
    if pattern == "lists overflow":
        s = lib.Sim(params, state, cell_lanes=0)
        s.step(1)
        i = [np.minimum((a * M).astype(np.int64), M - 1) for a in s.get_state()[:3]]
        s.close()
        now = np.bincount((i[0] * M + i[1]) * M + i[2], minlength=M ** 3)
        for c in (3, 100, 101, 6858):
            assert _filtered(int(now[c]), c, 0, params) > 300
    assert _fused_step_check(orc, lib, params, state, nsteps, 0, pattern) > 1000


@pytest.mark.parametrize("pattern", PATTERNS)
def test_group_counters(orc, lib, pattern):  # noqa: F811
    from paper_1208_0961_amd import batch
    from paper_1208_0961_amd import cuba as C
    occ = _occupancy(pattern)
    params = _params(occ, pattern)
    assert _takes_group_kernel(occ, params)
    state = _grid_state(occ, m=M)
    want = dict(pairs=0, candidates=0, claims=0)
    s = lib.Sim(params, state, cell_lanes=0)
    prev, profiles = state, []
    for t in range(2):
        st = orc.State(*prev)
        tr = orc.step(_orc_params(orc, params), st, t, trace=True)
        n = np.diff(tr["offsets"].astype(np.int64))
        want["pairs"] += int(np.sum(n * (n - 1) // 2))
        want["candidates"] += len(_rows(tr["cand"]))
        want["claims"] += len(_rows(tr["claim"]))
        s.step(1)
        prev = s.get_state()
        profiles.append(s.observe())
    single = C.cuba_counters(s.ctx)
    s.close()
    s = lib.Sim(params, state, cell_lanes=0)
    s.step(2)
    fused = C.cuba_counters(s.ctx)
    s.close()
    B = batch.Batch(1)
    B.admit(0, params, state)
    B.set_cell_lanes(0, 0)
    obs = B.set_observe(0, 1, rows=2)
    B.step(2)
    B.sync()
    assert list(single.values()) == list(want.values())
    assert single == fused == B.counters(0)
    for a, b in zip(B.get_state(0), prev):
        assert np.array_equal(a, b)
    tol = 2.0 * len(state[0]) * 2.0 ** -53      # two orders of a slab's sums
    for t, (T00, T0x) in enumerate(profiles):
        row = obs[(t + 1) % 2].cpu().numpy()
        assert np.all(np.abs(row[0] - T00) <= tol * T00)
        assert np.all(np.abs(row[1] - T0x) <= tol * T00)
    B.close()
