"""The health report of the adjoint's reverse sweep when it finds its levels
in the segment store instead of recomputing them: a trajectory that lost
positivity is reported by every sweep over it, reported before or not, and
only by those."""

import numpy as np
import pytest

from paper_1106_0785_amd import inputs

pytestmark = pytest.mark.gpu


# one segment, several, and levels stored by windows, by one workgroup and one by one
@pytest.mark.parametrize("nx,ny,steps,ckpt", [(20, 16, 6, 6), (64, 40, 6, 6), (64, 40, 7, 3), (520, 200, 4, 4)])
def test_lost_positivity_is_reported_by_every_sweep(nx, ny, steps, ckpt):
    import torch

    from paper_1106_0785_amd import lbm
    from paper_1106_0785_amd.autograd import Adjoint

    p, good = inputs.smooth_periodic(seed=4, nx=nx, ny=ny, amp=0.05)
    bad = {k: v.copy() for k, v in good.items()}
    bad["T"][ny // 2, nx // 3] = -0.5
    dev = [[torch.as_tensor(np.ascontiguousarray(f[k]), device="cuda") for k in ("rho", "ux", "uy", "T")]
           for f in (good, bad)]
    g = torch.ones((ny, nx), dtype=torch.float64, device="cuda")
    a = Adjoint(p, steps, ckpt_interval=ckpt)

    def refused(call):
        with pytest.raises(lbm.LbmError) as e:
            call()
        assert e.value.status == -5

    for _ in range(2):
        refused(lambda: a.forward(*dev[1]))
        refused(lambda: a.backward(g_rho=g))
        refused(lambda: a.backward(g_rho=g))
        a.forward(*dev[0])
        first = a.backward(g_rho=g)[0][0].clone()
        assert torch.equal(first, a.backward(g_rho=g)[0][0])
    a.close()
