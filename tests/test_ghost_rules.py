"""CPU check of the ghost-layer rule (host build of the kernels' own function)
against its definition, for every boundary kind, axis lengths from 1 (where a
two-deep periodic ghost wraps twice) and both ghost layers."""

import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "native", "ghost_host.cpp")
OUT = os.path.join(HERE, "native", "_build", "libghost_host.so")
CSRC = os.path.join(HERE, "..", "paper_1106_0785_amd", "csrc")
PERIODIC, ZERO_GRADIENT, SPECULAR, NEQ_WALL, FIXED = range(5)


@pytest.fixture(scope="module")
def lib():
    os.makedirs(os.path.dirname(OUT), exist_ok=True)
    newest = max(os.path.getmtime(p) for p in [SRC] + [os.path.join(CSRC, h) for h in os.listdir(CSRC)])
    if not os.path.exists(OUT) or os.path.getmtime(OUT) < newest:
        subprocess.check_call(["/opt/rocm/bin/hipcc", "--offload-arch=gfx950", "-O1", "-std=c++17", "-fPIC", "-shared",
                               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", SRC, "-o", OUT],
                              stderr=subprocess.DEVNULL)
    return ctypes.CDLL(OUT)


def expected(i, n, lo, hi, side_lo):
    if 0 <= i < n:
        return [i, 0, -1, PERIODIC]
    low = i < 0
    kind, side = (lo, side_lo) if low else (hi, side_lo + 1)
    if kind == PERIODIC:
        return [i % n, 0, side, kind]
    if kind == SPECULAR:  # about the wall half a spacing outside the end node
        return [min(-1 - i, n - 1) if low else max(2 * n - 1 - i, 0), 1, side, kind]
    return [0 if low else n - 1, 2 if kind == FIXED else 0, side, kind]


@pytest.mark.parametrize("n", [1, 2, 3, 5, 64])
def test_ghost_rule(lib, n):
    out = np.zeros(4, dtype=np.int32)
    for lo in range(5):
        for hi in range(5):
            for side_lo in (0, 2):
                for i in range(-2, n + 2):
                    lib.host_resolve(i, n, lo, hi, side_lo, out.ctypes.data_as(ctypes.c_void_p))
                    assert list(out) == expected(i, n, lo, hi, side_lo), (i, n, lo, hi, side_lo)
