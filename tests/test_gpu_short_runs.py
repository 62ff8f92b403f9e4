"""Calls of a few steps, and the last steps of longer ones, where a handle's
default kernel takes several steps per launch: the same states as the plain
kernel (the bound of the other kernels' comparisons) at the lines of the rule
that cuts a run into launches, and no slower than the one-step kernel."""

import numpy as np
import pytest

from gpu_util import gpu_run, log
from paper_1106_0785_amd import inputs
from test_gpu_parity import _kernel_diff

pytestmark = pytest.mark.gpu


def _problem(kind, nx, ny):
    if kind == "walls":
        return inputs.couette(0.7, nx=nx, ny=ny)[:2]
    if kind == "tube":
        return inputs.riemann("sod", nx=nx, ny=ny)[:2]
    return inputs.smooth_periodic(seed=5, nx=nx, ny=ny, amp=0.06)


# one workgroup, narrow grids with 12- and 8-step windows, up to 128 windows, more, and three rounds of them
@pytest.mark.parametrize("kind,nx,ny", [
    ("periodic", 16, 16), ("walls", 4, 64), ("tube", 700, 16), ("tube", 2000, 4), ("periodic", 128, 64),
    ("periodic", 136, 64), ("walls", 100, 100), ("periodic", 400, 300), ("periodic", 600, 256), ("walls", 600, 256)])
def test_calls_of_few_steps(kind, nx, ny):
    from paper_1106_0785_amd import lbm

    p, fl = _problem(kind, nx, ny)
    sim = lbm.Simulation(p)
    sim.init(**fl)
    done = 0
    for k in (1, 2, 3, 1, 5, 13):
        sim.step(k)
        done += k
        if done in (1, 3, 7, 25):
            _, ref = gpu_run(p, fl, done, variant=1)
            assert _kernel_diff(sim.get_f().cpu().numpy(), ref) <= 1e-13, done
    sim.check()
    sim.close()


@pytest.mark.parametrize("kind,nx,ny,steps,tuned", [
    ("periodic", 512, 128, 1, False), ("periodic", 768, 256, 1, False), ("walls", 1024, 256, 1, False),
    ("walls", 1024, 256, 2, False), ("periodic", 512, 128, 1, True), ("periodic", 768, 256, 1, True)])
def test_no_slower_than_the_one_step_kernel(kind, nx, ny, steps, tuned):
    """Both timed in turn; the margin (1.25) is several times the spread of such timings (a few percent), and the
    windowed kernel takes 1.4 to 2.5 times as long for these calls."""
    import torch

    from paper_1106_0785_amd import lbm

    p, fl = _problem(kind, nx, ny)
    sims = [lbm.Simulation(p), lbm.Simulation(p)]
    sims[1].set_variant(0)
    if tuned:  # (tuned by runs of 20 steps)
        sims[0].init(**fl)
        sims[0].tune(probe_steps=20)
    for s in sims:
        s.init(**fl)
        s.step(20)
    times = [[], []]
    for _ in range(7):
        for s, t in zip(sims, times):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(40):
                s.step(steps)
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b) / 40)
    chosen, one = (float(np.median(t)) for t in times)
    log("%s %dx%d step(%d): %s %.1f us, one-step kernel %.1f us" % (kind, nx, ny, steps, "tuned" if tuned else "default",
                                                                  1e3 * chosen, 1e3 * one))
    for s in sims:
        s.close()
    assert chosen <= 1.25 * one
