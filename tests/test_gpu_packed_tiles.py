"""Packed cells over the tile sizes that the box selects (4 to 64 cells a
workgroup, on both sides of the lines between them), a last tile that is not
full, and boxes of a dense and a sparse half: fused and collide-only steps
against one oracle step."""
import numpy as np
import pytest

from paper_1208_0961_amd import workload as W
from test_gpu_parity import lib  # noqa: F401
from test_gpu_small_cells import _fused_step_check

pytestmark = pytest.mark.gpu


# cells, mean (dense half, sparse half): tiles of 4, 8 (not 4), 8 / 16 (not 8),
# 8 (two units a wave), 32 (not 16), 64
@pytest.mark.parametrize("cells,dense,sparse", [
    ((41, 10, 9), 30, 30), ((99, 10, 10), 17, 17), ((111, 10, 9), 12, 11), ((105, 10, 10), 18, 2),
    ((41, 25, 25), 4, 4), ((101, 32, 29), 3, 1)])
@pytest.mark.parametrize("nsteps", (1, 2))
def test_packed_tile_sizes(orc, lib, cells, dense, sparse, nsteps):  # noqa: F811
    n_cells = int(np.prod(cells))
    box = tuple(c / 10.0 for c in cells)
    rng = np.random.default_rng(n_cells)
    half = (0.5 * box[0], box[1], box[2])
    parts = [W.sample_gas(rng, m * n_cells // 2, 0.4, (lo, 0, 0), (lo + half[0],) + half[1:])
             for m, lo in ((dense, 0.0), (sparse, half[0]))]
    perm = rng.permutation(sum(len(p[0]) for p in parts))
    state = [np.ascontiguousarray(np.concatenate(a)[perm]) for a in zip(*parts)]
    params = dict(box=box, cells=cells, sigma=0.02 * 1e-3 / 0.02, r_test=1.0, dt=0.02, seed=6)
    assert _fused_step_check(orc, lib, params, state, nsteps, 1, f"{cells} {dense}/{sparse}") > 500
