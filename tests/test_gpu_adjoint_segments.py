"""The adjoint's forward pass takes several steps per launch between
checkpoints and leaves the last segment's levels for the backward pass: the
final state is the time stepper's (bound as in the other kernels'
comparisons), and a second backward pass, which has to recompute that
segment, returns the same bits, also with other calls between."""

import numpy as np
import pytest

from paper_1106_0785_amd import inputs
from test_gpu_parity import _kernel_diff

pytestmark = pytest.mark.gpu


def _problem(kind, nx, ny):
    if kind == "walls":
        return inputs.couette(0.7, nx=nx, ny=ny)[:2]
    if kind == "rm":
        return inputs.rm(seed=2, nx=nx, ny=ny)[:2]
    return inputs.smooth_periodic(seed=5, nx=nx, ny=ny, amp=0.06)


# one workgroup, windows (with walls, narrow, several per CU), two steps per
# launch; segments of 1, several and all steps, and a short last one
@pytest.mark.parametrize("kind,nx,ny,steps,ckpt", [
    ("periodic", 20, 16, 11, 0), ("walls", 6, 60, 13, 5), ("walls", 30, 45, 14, 0), ("rm", 150, 7, 10, 4),
    ("rm", 130, 40, 17, 0), ("rm", 130, 40, 9, 9), ("rm", 130, 40, 4, 1), ("rm", 520, 400, 7, 3)])
def test_segments(kind, nx, ny, steps, ckpt):
    import torch

    from paper_1106_0785_amd import lbm
    from paper_1106_0785_amd.autograd import Adjoint

    p, fl = _problem(kind, nx, ny)
    dev = {k: torch.as_tensor(np.ascontiguousarray(v), device="cuda") for k, v in fl.items()}
    sim = lbm.Simulation(p)
    sim.init(**fl)
    sim.step(steps)
    ref = sim.moments()
    sim.close()
    adj = Adjoint(p, steps, ckpt_interval=ckpt)
    out = adj.forward(dev["rho"], dev["ux"], dev["uy"], dev["T"])
    a, b = (np.stack([m[k].cpu().numpy() for k in ("rho", "T")]) for m in (out, ref))
    assert _kernel_diff(a, b) <= 1e-13
    g = torch.sin(torch.arange(nx * ny, dtype=torch.float64, device="cuda")).reshape(ny, nx)

    def flat(r):
        return torch.cat([t.flatten() for t in (list(r[0]) if isinstance(r[0], (list, tuple)) else [r[0]]) + list(r[1:])])

    first = flat(adj.backward(g_rho=g, g_T=0.3 * g)).clone()
    assert bool(torch.isfinite(first).all())
    second = flat(adj.backward(g_rho=g, g_T=0.3 * g)).clone()
    assert torch.equal(first, second)
    adj.forward(dev["rho"], dev["ux"], dev["uy"], dev["T"])
    assert torch.equal(first, flat(adj.backward(g_rho=g, g_T=0.3 * g)))


# either side of the lines between the gather and the LDS-staged step, whose
# tiles are 4 rows tall in the second and 8 in the third
@pytest.mark.parametrize("nx,ny", [(512, 128), (400, 200), (512, 256), (513, 257)])
def test_both_steps_at_the_lines_of_their_rule(nx, ny):
    import torch

    from paper_1106_0785_amd.autograd import Adjoint

    p, fl = _problem("rm", nx, ny)
    dev = [torch.as_tensor(np.ascontiguousarray(fl[k]), device="cuda") for k in ("rho", "ux", "uy", "T")]
    g = torch.cos(torch.arange(nx * ny, dtype=torch.float64, device="cuda")).reshape(ny, nx)
    res = []
    for variant in (None, 0, 1):
        a = Adjoint(p, 5, 3)
        if variant is not None:
            a.set_variant(variant)
        a.forward(*dev)
        grads, gs = a.backward(g_rho=g)
        res.append([t.clone() for t in grads] + [gs.clone()])
        a.close()
    for other in res[1:]:
        for x, y in zip(res[0], other):
            assert float((x - y).abs().max()) <= 1e-12 * float(y.abs().max())
