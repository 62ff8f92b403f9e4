"""The windowed kernel (and the one-workgroup form of it) gives the plain
kernel's results bit by bit: the same node arithmetic in the same order, with
every kind of side, fixed states included (their ghosts' velocities come from
the host)."""

import numpy as np
import pytest

from gpu_util import gpu_run
from paper_1106_0785_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(20, 16), (150, 7), (90, 61)])
@pytest.mark.parametrize("bc", [("periodic",) * 4, ("specular", "zero_gradient", "specular", "specular"),
                                ("neq_wall", "neq_wall", "periodic", "periodic"),
                                ("dirichlet_eq", "zero_gradient", "specular", "dirichlet_eq")])
@pytest.mark.parametrize("version", [1, 2, 3])
def test_same_bits(nx, ny, bc, version):
    p, f = inputs.smooth_periodic(seed=5, nx=nx, ny=ny, amp=0.05)
    p["bc"], p["eq_version"] = list(bc), version
    for side in range(4):
        p["wall"][side] = [1.03, 0.08, -0.04, 1.01]
    _, plain = gpu_run(p, f, 25, variant=1)
    _, windows = gpu_run(p, f, 25, variant=2 if nx * ny <= 512 else 3)
    assert np.array_equal(windows, plain)
