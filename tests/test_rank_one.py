"""CPU check (host build of the kernel's own functions) of when a matrix
power counts as rank one: X^2 = mu X up to 2^-44 |mu| |o|, o the entry the
two are compared through, for every multiple of X alike."""

import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "native", "rank_host.cpp")
OUT = os.path.join(HERE, "native", "_build", "librank_host.so")
CSRC = os.path.join(HERE, "..", "paper_1106_0785_amd", "csrc")
TOL = 2.0**-44


@pytest.fixture(scope="module")
def lib():
    os.makedirs(os.path.dirname(OUT), exist_ok=True)
    newest = max(os.path.getmtime(p) for p in [SRC] + [os.path.join(CSRC, h) for h in os.listdir(CSRC)])
    if not os.path.exists(OUT) or os.path.getmtime(OUT) < newest:
        subprocess.check_call(["/opt/rocm/bin/hipcc", "--offload-arch=gfx950", "-O1", "-std=c++17", "-fPIC", "-shared",
                               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", SRC, "-o", OUT],
                              stderr=subprocess.DEVNULL)
    return ctypes.CDLL(OUT)


def _verdict(lib, X, A, top):
    x, a = (np.ascontiguousarray(m.ravel()).view(np.float64) for m in (X, A))
    return bool(lib.host_rank_one(x.ctypes.data_as(ctypes.c_void_p), a.ctypes.data_as(ctypes.c_void_p), X.size, int(top)))


# what is left beside mu X, as a multiple of the bound; X's scale is a power
# of two, so that scaling commits no rounding
@pytest.mark.parametrize("left,within", [(0.25, True), (0.7, True), (1.6, False), (4.0, False)])
@pytest.mark.parametrize("scale", [-40, -6, -1, 0, 1, 5, 20])
def test_bound_at_every_scale(lib, left, within, scale):
    for seed in range(6):
        rng = np.random.default_rng(seed)
        X = rng.uniform(-1, 1, (16, 16)) + 1j * rng.uniform(-1, 1, (16, 16))
        top = int(np.argmax(np.abs(X)))
        X = X * (1.0 / np.abs(X.flat[top]))
        mu = 3.0 + 0.5j
        A = mu * X
        other = (top + 37) % X.size
        A.flat[other] += left * TOL * np.abs(A.flat[top])  # a real step: |component| is the modulus
        s = 2.0**scale
        assert _verdict(lib, s * X, s * s * A, top) == within, (seed, scale, left)
