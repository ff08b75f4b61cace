"""Boxes of 6000 cells and more with means around 50 and 110 and few filtered
pairs, most of which take the kernel in which four cells share their pairs
(test_gpu_group_lists.py asserts that its boxes do, and overflows the lists):
groups past the last cell, cells whose list of filtered pairs is long and cells
past their block (each then taken by its own wave), fused and collide-only
steps against one oracle step, and a batched event against the lone run.  And
cells that outgrow the small LDS inside a block that holds them."""
import numpy as np
import pytest

from test_gpu_parity import lib  # noqa: F401
from test_gpu_small_cells import _fused_step_check, _grid_state

pytestmark = pytest.mark.gpu

M = 19   # 6859 cells: the last group holds 3


def _occupancy(pattern, seed=1):
    rng = np.random.default_rng(seed)
    occ = rng.poisson(112 if pattern == "long lists" else 52, M ** 3)
    if pattern == "long lists":       # sorted and resolved cell by cell
        occ[[5, 6, 7, 500]] = (20, 0, 290, 330)
    if pattern == "ragged":
        occ[::5] = rng.integers(0, 4, len(occ[::5]))
        occ[1::5] = 85
    if pattern == "lists overflow":
        occ[[3, 100, 6858]] = (260, 200, 180)
    if pattern == "blocks overflow":
        occ[[0, 77, 6857]] = (300, 140, 700)
    return occ


def _params(occ, scale=1.0):
    """K mean^2 = 9 scale at the grid's cells."""
    mean = float(np.mean(occ))
    vcell = 1.0 / M ** 3
    return dict(box=(1.0, 1.0, 1.0), cells=(M, M, M), r_test=1.0, dt=0.002,
                sigma=9.0 * scale / mean ** 2 * vcell / 0.002, seed=17, cell_capacity=128)


@pytest.mark.parametrize("nsteps", (1, 2))
@pytest.mark.parametrize("pattern", ("poisson", "ragged", "lists overflow", "blocks overflow",
                                     "long lists"))
def test_group_parity(orc, lib, pattern, nsteps):  # noqa: F811
    occ = _occupancy(pattern)
    long = pattern == "long lists"    # ~50 filtered pairs a cell, 400 in the fullest
    params = {**_params(occ, 3.0 if long else 1.0),
              "cell_capacity": 512 if long or pattern == "lists overflow" else 128}
    claims = _fused_step_check(orc, lib, params, _grid_state(occ, m=M), nsteps, 0, pattern)
    assert claims is None or claims > 1000


@pytest.mark.parametrize("pattern", ("poisson", "blocks overflow"))
def test_group_batch_equals_lone_run(lib, pattern):  # noqa: F811
    from paper_1208_0961_amd import batch
    occ = _occupancy(pattern, seed=3)
    state = _grid_state(occ, m=M, seed=4)
    small = _grid_state(np.full(8 ** 3, 3), m=8)
    B = batch.Batch(2)
    B.admit(0, _params(occ), state)
    B.admit(1, {**_params(occ), "cells": (8, 8, 8)}, small)
    obs = B.set_observe(0, 2, rows=2)
    B.step(4)
    B.sync()
    s = lib.Sim(_params(occ), state, cell_lanes=0)
    s.step(2)
    first = s.observe()
    s.step(2)
    second = s.observe()
    ref = s.get_state()
    s.close()
    for a, b in zip(B.get_state(0), ref):
        assert np.array_equal(a, b)
    got = obs.cpu().numpy()
    for row, want in ((1, first), (0, second)):
        assert np.allclose(got[row][0], want[0], rtol=1e-12, atol=0)
        assert np.allclose(got[row][1], want[1], rtol=1e-12, atol=1e-12 * np.abs(want[0]).max())
    B.close()


def test_cells_outgrow_the_small_lds(orc, lib):  # noqa: F811
    # 3 x 300 particles in blocks of 1024 stream into the middle cell
    rng = np.random.default_rng(5)
    n = 300
    x = np.concatenate([0.9 - 0.5 * rng.random(n), 1.2 + 0.5 * rng.random(n),
                        2.1 + 0.5 * rng.random(n)])
    pos = [x, rng.random(3 * n), rng.random(3 * n)]
    p = rng.normal(size=(3 * n, 3)) * 0.02
    p[:n, 0], p[n:2 * n, 0], p[2 * n:, 0] = 1.0, 0.0, -1.0
    state = [np.ascontiguousarray(a) for a in (*pos, *p.T)]
    params = dict(box=(3.0, 1.0, 1.0), cells=(3, 1, 1), sigma=1e-4, r_test=1.0, dt=0.06,
                  seed=23, cell_capacity=1024)
    for nsteps in (9, 10):
        sim = lib.Sim(params, state, cell_lanes=0)
        sim.step(nsteps - 1)
        mid = np.floor(sim.get_state()[0])
        sim.close()
        assert np.sum(mid == 1) > 512
        _fused_step_check(orc, lib, params, state, nsteps, 0, "outgrown")
