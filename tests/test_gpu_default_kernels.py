"""The kernel and shape a handle starts with, at the lines of the rules that
choose them, against the plain kernel (same node arithmetic; the bound is
that of the other kernels' comparisons) and, on small grids, the oracle."""

import pytest

from gpu_util import assert_parity, gpu_run, oracle_run
from paper_1106_0785_amd import inputs
from test_default_windows import default_window
from test_gpu_parity import _kernel_diff
from test_window_geometry import NEQ, PER

pytestmark = pytest.mark.gpu


def _problem(kind, nx, ny):
    if kind == "walls":
        return inputs.couette(0.7, nx=nx, ny=ny)[:2]
    p, fl = inputs.smooth_periodic(seed=5, nx=nx, ny=ny, amp=0.06)
    if kind == "limited":
        p["scheme"] = 1
    return p, fl


def _against_plain(p, fl, steps, setup=None):
    from paper_1106_0785_amd import lbm

    sim = lbm.Simulation(p)
    if setup:
        setup(sim)
    chosen = sim.variant(), sim.window()
    sim.init(**fl)
    sim.step(steps)
    out = {k: v.cpu().numpy() for k, v in sim.moments().items()}
    f = sim.get_f().cpu().numpy()
    sim.check()
    sim.close()
    _, f1 = gpu_run(p, fl, steps, variant=1)
    assert _kernel_diff(f, f1) <= 1e-13
    return out, chosen


# one workgroup per CU with each of the three shapes, several per CU, and both
# narrow rules
@pytest.mark.parametrize("kind,nx,ny", [
    ("periodic", 31, 17), ("periodic", 128, 128), ("periodic", 129, 128), ("walls", 130, 96), ("periodic", 520, 100),
    ("periodic", 521, 110), ("walls", 17, 300), ("periodic", 129, 4), ("periodic", 700, 16), ("periodic", 6200, 16)])
def test_default_window(kind, nx, ny):
    p, fl = _problem(kind, nx, ny)
    out, (variant, shape) = _against_plain(p, fl, 15)
    by = (NEQ, NEQ) if kind == "walls" else (PER, PER)
    w = default_window(nx, ny, (PER, PER), by)
    assert variant == 3 and shape == (min(w[0], nx), min(w[1], ny), w[2])
    if nx * ny <= 20000:
        assert_parity(out, oracle_run(p, fl, 15)[0], what="default window %s %dx%d" % (kind, nx, ny))


@pytest.mark.parametrize("kind,nx,ny,variant", [
    ("periodic", 768, 256, 3), ("periodic", 769, 256, 4), ("walls", 1024, 256, 3), ("walls", 1025, 256, 0),
    ("limited", 300, 200, 0), ("limited", 1023, 257, 0), ("periodic", 1500, 301, 4)])
def test_default_kernel(kind, nx, ny, variant):
    p, fl = _problem(kind, nx, ny)
    _, chosen = _against_plain(p, fl, 7)
    assert chosen[0] == variant


@pytest.mark.parametrize("kind", ["periodic", "walls"])
def test_window_of_384_nodes(kind):
    p, fl = _problem(kind, 90, 61)
    _against_plain(p, fl, 15, lambda s: (s.set_variant(3), s.set_window(24, 16, 4)))
