"""cuba_get_state of states large enough for its two-launch export: it leaves
the state as it was (the steps that follow are those of a run without it,
also where cells overflow their blocks), and a captured export replayed when
the buffer that it reads holds no state writes nothing and reads no slot."""
import numpy as np
import pytest

from paper_1208_0961_amd import workload as W
from test_gpu_parity import lib  # noqa: F401

pytestmark = pytest.mark.gpu

N = 131072 + 77
BOX, CELLS = (10.0, 2.0, 2.0), (16, 4, 4)


def _params(sigma, cap):
    return dict(box=BOX, cells=CELLS, sigma=sigma, r_test=100.0, dt=0.01, seed=5,
                cell_capacity=cap)


@pytest.mark.parametrize("cap", (64, 1024))   # blocks of a tenth, all of a cell's particles
def test_steps_after_an_export(lib, cap):  # noqa: F811
    state = W.thermal_box(BOX, N, 0.4, seed=3)
    a, b = lib.Sim(_params(0.02, cap), state), lib.Sim(_params(0.02, cap), state)
    for k in (3, 2):
        a.step(k)
        a.get_state()
    b.step(5)
    moved = 0
    for u, v, w in zip(a.get_state(), b.get_state(), state):
        assert np.array_equal(u, v)
        moved += int((u != w).sum())
    assert moved > 2 * N
    a.close()
    b.close()


@pytest.mark.parametrize("cap", (64, 1024))
def test_streamed_positions_under_their_ids(orc, lib, cap):  # noqa: F811
    state = W.thermal_box(BOX, N, 0.4, seed=4)
    s = lib.Sim(_params(0.0, cap), state)
    s.step(3)
    got = s.get_state()
    s.close()
    st = orc.State(*state)
    p = {k: v for k, v in _params(0.0, cap).items() if k != "cell_capacity"}
    orc.run(orc.make_params(**p), st, 0, 3, 8)
    for d in range(6):
        assert np.array_equal(got[d], st[d])


def test_replayed_export_of_the_other_buffer(lib):  # noqa: F811
    import torch
    from paper_1208_0961_amd import cuba as C
    state = W.thermal_box(BOX, N, 0.4, seed=5)
    stream = torch.cuda.Stream()
    ref = lib.Sim(_params(0.02, 1024), state)
    ref.step(2)
    two = ref.get_state()
    ref.step(1)
    three = ref.get_state()
    ref.close()
    with torch.cuda.stream(stream):
        s = lib.Sim(_params(0.02, 1024), state, stream=stream)
        out = torch.empty((6, s.n), dtype=torch.float64, device="cuda")
        stream.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            C.cuba_get_state(s.ctx, *[out[d].data_ptr() for d in range(6)])
        s.step(1)           # the state is in the other buffer, nothing was ever listed
        g.replay()          # (outputs unspecified)
        s.step(1)
        g.replay()
        stream.synchronize()
        got_two = out.cpu().numpy()
        s.step(1)
        g.replay()
        got_three = s.get_state()
        s.close()
    for d in range(6):
        assert np.array_equal(got_two[d], two[d])
        assert np.array_equal(got_three[d], three[d])
