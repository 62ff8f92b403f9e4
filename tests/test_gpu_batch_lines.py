"""Line instances of a batch at the edges of a region (128 and 256 nodes),
along both axes, with every boundary kind at either end (the ghost entries
beside a region hold them), against the oracle. Tolerance: the per-field
parity bound of every GPU test (1e-11)."""

import pytest

from gpu_util import assert_parity, oracle_run
from paper_1106_0785_amd import inputs

pytestmark = pytest.mark.gpu

ENDS = [("zero_gradient", "specular"), ("dirichlet_eq", "zero_gradient"), ("specular", "dirichlet_eq"),
        ("neq_wall", "neq_wall"), ("neq_wall", "specular"), ("periodic", "periodic")]
SIZES = [2, 3, 31, 127, 128, 129, 255, 256, 257, 450]


def _line(n, axis, ends, version):
    nx, ny = (n, 1) if axis == 0 else (1, n)
    p, f = inputs.smooth_periodic(seed=n + axis, nx=nx, ny=ny, eq_version=version)
    p["bc"] = list(ends) + ["periodic"] * 2 if axis == 0 else ["periodic"] * 2 + list(ends)
    for side, (rho, ux, uy, T) in enumerate([(1.03, 0.08, -0.04, 1.01), (0.98, 0.12, -0.06, 0.99)] * 2):
        p["wall"][side] = [rho, ux, uy, T]
    return p, f


@pytest.mark.parametrize("region,h,persistent", [(128, 16, True), (256, 24, False)])
def test_lines_with_every_end(region, h, persistent):
    from paper_1106_0785_amd.batch import Batch

    items = []
    for axis in (0, 1):
        for k, ends in enumerate(ENDS):
            for n in SIZES:
                if "neq_wall" in ends and n < 3:
                    continue
                items.append(_line(n, axis, ends, 1 + (k + n) % 2))
    b = Batch([p for p, _ in items])
    b.set_schedule(region, h)
    b.set_persistent(persistent)
    b.init([f for _, f in items])
    b.step(37)
    b.check()
    m = {k: v.cpu().numpy() for k, v in b.moments().items()}
    for i, (p, f) in enumerate(items):
        o, _ = oracle_run(p, f, 37)
        assert_parity({k: b.split(v, i) for k, v in m.items()}, o,
                      what="line %d x %d, %s" % (p["nx"], p["ny"], p["bc"]))
    b.close()
