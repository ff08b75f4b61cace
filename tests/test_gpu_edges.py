"""Streaming and cell indices where the shared-reciprocal velocity and the
reciprocal cell index hand over to divisions: positions at and within a few
ulps of every cell face, components of zero, and momenta at both ends of the
range the shared reciprocal takes.  One traced step without collisions
against the oracle: cells, positions and momenta bit for bit."""
import numpy as np
import pytest

from test_gpu_parity import compare_step, lib  # noqa: F401

pytestmark = pytest.mark.gpu


def _faces(L, n):
    """Every face of an axis and its neighbours up to 3 ulps, inside [0, L]."""
    q = np.minimum(np.arange(n + 1) * (L / n), L)
    out = [q]
    lo = hi = q
    for _ in range(3):
        lo, hi = np.nextafter(lo, -1.0), np.nextafter(hi, 2 * L)
        out += [lo, hi]
    q = np.concatenate(out)
    return q[(q >= 0.0) & (q <= L)]


def _state(box, cells, seed=11):
    rng = np.random.default_rng(seed)
    pos, mom = [], []
    for d in range(3):        # at rest along d, on the faces of axis d
        q = _faces(box[d], cells[d])
        r = rng.random((len(q), 3)) * np.asarray(box)
        r[:, d] = q
        p = rng.normal(size=(len(q), 3))
        p[:, d] = 0.0
        pos.append(r)
        mom.append(p)
    m = 400                   # whole vectors and single components rescaled
    for e in (-505, -500, -499, -300, 0, 249, 250, 251, 400):
        pos.append(rng.random((m, 3)) * np.asarray(box))
        mom.append(rng.normal(size=(m, 3)) * 2.0 ** e)
    for e in (-1060, -800, -501, -500, -499, -60):
        p = rng.normal(size=(m, 3))
        p[np.arange(m), rng.integers(0, 3, m)] *= 2.0 ** e
        pos.append(rng.random((m, 3)) * np.asarray(box))
        mom.append(p)
    r, p = np.concatenate(pos), np.concatenate(mom)
    return [np.ascontiguousarray(a) for a in (*r.T, *p.T)]


@pytest.mark.parametrize("lanes", (0, 1, 16))
@pytest.mark.parametrize("box,cells", [((10.0, 1.0, 3.0), (100, 7, 13)),
                                       ((6.4, 1.0, 1.0), (64, 1, 3))])
def test_faces_and_extreme_momenta(orc, lib, lanes, box, cells):  # noqa: F811
    params = dict(box=box, cells=cells, sigma=0.0, r_test=10.0, dt=0.03, seed=3)
    state = _state(box, cells)
    for t in range(2):
        state, _ = compare_step(orc, lib, params, state, t, "edges", lanes=lanes)
