"""GPU parity of the stencil's default form (AUTO) with the oracle, bit for
bit, where the shape decides: every width of the windows, a caller's workgroup
size or grid, and a caller's graph."""
import sys

import numpy as np
import pytest

import oracle
from paper_2004_05371_amd import inputs
from test_stencil_plan import WIDTHS

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def run(lib, x, steps, r, grid=0, wg=0, shift=0):
    base = torch.zeros(x.size + 8, dtype=torch.float32, device="cuda")
    u = base[shift:shift + x.size]
    u.copy_(torch.from_numpy(x))
    scratch = torch.full((x.size,), float("nan"), dtype=torch.float32, device="cuda")
    opts = lib.make_opts(variant=0, wg=wg, grid=grid)
    lib.stencil_jacobi_1d(u.data_ptr(), scratch.data_ptr(), x.size, steps, r, 0, lib.current_stream(), opts)
    torch.cuda.synchronize()
    assert lib.red_check_error(lib.current_stream()) == lib.RED_OK
    return u.cpu().numpy()


@pytest.mark.parametrize("v", sorted(WIDTHS))
def test_blocked_steps_every_window_width(lib, v):
    """Each width of the windows that AUTO takes, aligned and not."""
    n, steps = WIDTHS[v]
    x = inputs.normal_f32(n, sub=82)
    say("window width", v, n, steps)
    want = oracle.jacobi_1d_f32(x, steps, 0.25)
    for shift in (0, 1, 3):
        got = run(lib, x, steps, 0.25, shift=shift)
        assert np.array_equal(got, want), (v, n, steps, shift, np.flatnonzero(got != want)[:5])


@pytest.mark.parametrize("n,wg,grid", [(100_003, 256, 0), (100_003, 0, 32), (4099, 64, 4), (12_000_001, 512, 0),
                                       (12_000_001, 0, 256)])
def test_auto_with_a_callers_shape(lib, n, wg, grid):
    """AUTO with a workgroup size or a grid: the persistent form where the
    windows fit the chip, else one launch per step, bit for bit."""
    x = inputs.normal_f32(n, sub=83)
    steps = 3 if n > 1_000_000 else 40
    want = oracle.jacobi_1d_f32(x, steps, 0.25)
    say("auto with a shape", n, wg, grid)
    got = run(lib, x, steps, 0.25, wg=wg, grid=grid)
    assert np.array_equal(got, want), (n, wg, grid, np.flatnonzero(got != want)[:5])


@pytest.mark.parametrize("n,steps", [(300, 7), (300_007, 130), (4_194_305, 2)])
def test_auto_in_a_graph(lib, n, steps):
    """AUTO recorded into a caller's graph (one window, blocked steps, one
    launch per step) and replayed: each replay continues from the state before
    it, with the program's own eager call in between."""
    x = inputs.normal_f32(n, sub=84)
    u = torch.from_numpy(x).to("cuda")
    sc = torch.empty_like(u)
    torch.cuda.synchronize()
    st = torch.cuda.Stream()

    def step():
        lib.stencil_jacobi_1d(u.data_ptr(), sc.data_ptr(), n, steps, 0.3, 0, st.cuda_stream)
    step()
    st.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        step()
    want = oracle.jacobi_1d_f32(x, steps, 0.3)
    assert np.array_equal(u.cpu().numpy(), want)
    for rep in range(4):
        say("auto replay", n, steps, rep)
        g.replay()
        torch.cuda.synchronize()
        want = oracle.jacobi_1d_f32(want, steps, 0.3)
        assert np.array_equal(u.cpu().numpy(), want), rep
        step()
        torch.cuda.synchronize()
        want = oracle.jacobi_1d_f32(want, steps, 0.3)
        assert np.array_equal(u.cpu().numpy(), want), rep
