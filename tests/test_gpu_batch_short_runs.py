"""Batches in the persistent form of the line kernel: calls of one block take
a plain launch. The same bits as with a launch per block, on calls around the
length of a block and in sequence (both buffers' turns), versions 1 and 3 at
both regions; and no slower than those for a single step."""

import numpy as np
import pytest

from gpu_util import log
from paper_1106_0785_amd import inputs

pytestmark = pytest.mark.gpu


def _batch(version, n):
    from paper_1106_0785_amd.batch import Batch

    items = inputs.batch(seed=6, n=n, riemann_n=(200, 1500), couette_h=(32, 200))
    b = Batch([dict(p, eq_version=version) for _, p, _ in items])
    b.init([f for _, _, f in items])
    return b


@pytest.mark.parametrize("version", [1, 3])
@pytest.mark.parametrize("region,h", [(128, 12), (256, 16)])
@pytest.mark.parametrize("graph", [False, True])
def test_same_bits(version, region, h, graph):
    out = []
    for persistent in (False, True):
        b = _batch(version, 12)
        b.set_schedule(region, h, graph)
        b.set_persistent(persistent)
        states = []
        for k in (1, h - 1, h, h + 1, 1, 3 * h + 2, 2):
            b.step(k)
            states.append(b.get_f().cpu().numpy())
        b.check()
        b.close()
        out.append(states)
    for a, c in zip(*out):
        assert np.array_equal(a, c)


@pytest.mark.parametrize("version", [1, 3])
def test_single_step_no_slower_than_a_launch_per_block(version):
    """Timed in turn; the margin (1.25) is several times the spread, and the persistent launch took three times as
    long for one step."""
    import torch

    b = _batch(version, 200)
    b.set_schedule(256, 16)
    times = {False: [], True: []}
    for _ in range(7):
        for persistent in (False, True):
            b.set_persistent(persistent)
            b.step(1)
            b.step(1)
            s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            s.record()
            for _ in range(30):
                b.step(1)
            e.record()
            e.synchronize()
            times[persistent].append(s.elapsed_time(e) / 30)
    b.close()
    blocks, pers = (float(np.median(times[k])) for k in (False, True))
    log("one step of 200 lines, version %d: launch per block %.1f us, persistent %.1f us" % (version, 1e3 * blocks, 1e3 * pers))
    assert pers <= 1.25 * blocks
