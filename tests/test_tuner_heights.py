"""The tile heights that lbm_tune times (host function of the library, no
GPU): ascending, each once, the handle's own among them, whether or not it is
one of the fixed list (default tiles may be 36, 44, 52 or 60 rows)."""

import ctypes

import numpy as np
import pytest


@pytest.mark.parametrize("start", [4, 6, 36, 44, 52, 60, 64, 70, 300, 1024])
def test_heights(start):
    from paper_1106_0785_amd import lbm

    fn = lbm.load()._ZN3lbm12tile_heightsEiPi  # lbm::tile_heights(int, int*)
    fn.argtypes, fn.restype = [ctypes.c_int, ctypes.c_void_p], ctypes.c_int
    out = np.full(32, -1, dtype=np.int32)
    n = fn(start, out.ctypes.data_as(ctypes.c_void_p))
    heights = list(out[:n])
    assert start in heights and heights == sorted(set(heights)) and list(out[n:]) == [-1] * (32 - n)
    assert set(heights) - {start} <= {4, 8, 12, 16, 20, 24, 28, 32, 40, 48, 56, 64, 96, 128, 192, 256}
    assert n in (16, 17)
