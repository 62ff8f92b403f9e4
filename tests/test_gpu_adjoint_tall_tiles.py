"""The adjoint step on tiles that march many rows, against the gather step.

901 x 603 gives the LDS-staged step tiles of 20 rows, five iterations of its
march, with a ragged last tile (3 rows) and last strip (33 of 62 columns): from
the third iteration on a wave takes f^n from the rows handed on in LDS
(versions 1 and 2) or reads it again (version 3). The gather step takes its
two-blocks-per-CU form there (2265 blocks, versions 1 and 2). Bound of the
gradients of the fields: the two forms' other comparison, 1e-12 of each one's
largest value. The rates' gradients are sums over all nodes, in another order
in each form and with terms of both signs, so rounding has no such bound: what
is held is that every node is in the sum. The shock/interface problem is used
for that, with one seed of one sign; a tile left out changes the sums by a
465th on average, and cancellation by a factor of up to 1e6 would leave their
rounding below 1e-8: bound 1e-6."""

import numpy as np
import pytest

from paper_1106_0785_amd import inputs

pytestmark = pytest.mark.gpu

NX, NY = 901, 603


def _problem(kind, version):
    if kind == "walls":
        p, f = inputs.couette(0.7, nx=NX, ny=NY)[:2]
        x = (np.arange(NX) + 0.5) / NX
        y = np.arange(NY)[:, None] / (NY - 1)
        f["uy"] = f["uy"] + 0.03 * np.sin(2 * np.pi * x)[None, :] * np.sin(np.pi * y) ** 2
    else:
        p, f = inputs.smooth_periodic(seed=8, nx=NX, ny=NY, amp=0.06)
        if kind == "open":
            p["bc"] = ["dirichlet_eq", "zero_gradient", "specular", "zero_gradient"]
            p["wall"][0] = [1.03, 0.08, -0.04, 1.01]
    p["eq_version"] = version
    return p, f


@pytest.mark.parametrize("kind", ["periodic", "open", "walls"])
@pytest.mark.parametrize("version", [1, 2, 3])
def test_staged_against_gather(kind, version):
    import torch

    from paper_1106_0785_amd.autograd import Adjoint

    p, f = _problem(kind, version)
    dev = [torch.as_tensor(np.ascontiguousarray(f[k]), device="cuda") for k in ("rho", "ux", "uy", "T")]
    k = torch.arange(NX * NY, dtype=torch.float64, device="cuda").reshape(NY, NX)
    seeds = [torch.sin(0.7 * k), torch.cos(0.3 * k), torch.sin(0.11 * k), torch.cos(1.3 * k)]
    res = []
    for variant in (0, 1):
        a = Adjoint(p, 3, 2)
        a.set_variant(variant)
        a.forward(*dev)
        grads, gs = a.backward(*seeds)
        res.append([t.clone() for t in grads] + [gs.clone()])
        a.close()
    for x, y in zip(res[0][:4], res[1][:4]):
        assert float((x - y).abs().max()) <= 1e-12 * float(y.abs().max())


@pytest.mark.parametrize("version", [1, 2, 3])
def test_every_node_is_in_the_rates_gradient(version):
    import torch

    from paper_1106_0785_amd.autograd import Adjoint

    p, f = inputs.rm(seed=2, nx=NX, ny=NY)[:2]
    p["eq_version"] = version
    dev = [torch.as_tensor(np.ascontiguousarray(f[k]), device="cuda") for k in ("rho", "ux", "uy", "T")]
    res = []
    for variant in (0, 1):
        a = Adjoint(p, 3, 2)
        a.set_variant(variant)
        a.forward(*dev)
        res.append(a.backward(g_rho=dev[0])[1].clone())
        a.close()
    assert float(res[1].abs().max()) > 0.0
    assert float((res[0] - res[1]).abs().max()) <= 1e-6 * float(res[1].abs().max())
