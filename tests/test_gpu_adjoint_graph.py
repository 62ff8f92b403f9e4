"""Adjoint calls captured into HIP graphs through the C ABI: the library does
not see a replay overwrite the segment store, so a handle that has seen a
capture must not take stored levels for those of its last forward call. Every
gradient is compared bit by bit with a fresh handle's."""

import ctypes

import numpy as np
import pytest

from paper_1106_0785_amd import inputs

pytestmark = pytest.mark.gpu

NX, NY, STEPS = 150, 40, 7


class _Calls:
    """A handle on a stream of its own, with buffers that graphs may refer to."""

    def __init__(self, p, ckpt):
        import torch

        from paper_1106_0785_amd import autograd

        self.lib = autograd._lib()
        self.stream = torch.cuda.Stream()
        with torch.cuda.stream(self.stream):
            self.adj = autograd.Adjoint(p, STEPS, ckpt)
        new = lambda: torch.zeros((NY, NX), dtype=torch.float64, device="cuda")
        self.fields = [new() for _ in range(4)]
        self.seed = torch.sin(torch.arange(NX * NY, dtype=torch.float64, device="cuda")).reshape(NY, NX)
        self.grads = [new() for _ in range(4)]
        self.grad_s = torch.zeros(16, dtype=torch.float64, device="cuda")

    def _p(self, t):
        return ctypes.c_void_p(t.data_ptr())

    def forward(self):
        assert self.lib.lbm_adjoint_forward(self.adj.handle, *map(self._p, self.fields)) == 0

    def backward(self):
        assert self.lib.lbm_adjoint_backward(self.adj.handle, *map(self._p, self.fields), self._p(self.seed), None, None,
                                             None, *map(self._p, self.grads), self._p(self.grad_s)) == 0

    def capture(self, call):
        import torch

        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=self.stream):
            call()
        return g

    def run(self, what, fields=None):
        """An eager call or a replay; the result of a backward one."""
        import torch

        torch.cuda.synchronize()
        if fields is not None:
            for t, f in zip(self.fields, fields):
                t.copy_(f)
        torch.cuda.synchronize()
        with torch.cuda.stream(self.stream):
            what.replay() if hasattr(what, "replay") else what()
        torch.cuda.synchronize()
        return torch.cat([t.flatten() for t in self.grads] + [self.grad_s]).clone()


# one segment and several
@pytest.mark.parametrize("ckpt", [0, STEPS])
def test_replays_and_eager_calls(ckpt):
    import torch

    p = inputs.rm(seed=2, nx=NX, ny=NY)[0]
    sets = [[torch.as_tensor(np.ascontiguousarray(inputs.rm(seed=s, nx=NX, ny=NY)[1][k]), device="cuda")
             for k in ("rho", "ux", "uy", "T")] for s in (2, 3, 4)]
    want = []
    for f in sets:
        fresh = _Calls(p, ckpt)
        fresh.run(fresh.forward, f)
        want.append(fresh.run(fresh.backward))
        fresh.adj.close()
    assert not torch.equal(want[0], want[1])

    c = _Calls(p, ckpt)
    c.run(c.forward, sets[0])  # eager: its levels stay stored
    back = c.capture(c.backward)
    c.run(c.forward, sets[1])
    assert torch.equal(c.run(back), want[1])
    fwd = c.capture(c.forward)
    for a, b in ((0, 1), (2, 0), (1, 2)):
        c.run(c.forward, sets[a])  # eager on one set,
        c.run(fwd, sets[b])        # a replay on another
        assert torch.equal(c.run(c.backward), want[b])
        c.run(fwd, sets[a])
        assert torch.equal(c.run(back), want[a])
        assert torch.equal(c.run(c.backward), want[a])
    c.adj.close()
