"""The tiles of the explicit step with 8 points per cell, from the library's own rule (host code, no GPU): within a
block's threads, covering the mesh, and as deep as was measured best (within 6 %) at the edges that were timed."""
import ctypes as C
import os

import pytest

H = pytest.importorskip("paper_1009_0457_amd.hmc")
if not os.path.exists(H.LIB_PATH):
    pytest.skip("libhmc.so not built", allow_module_level=True)


def tile(K):
    f = getattr(C.CDLL(H.LIB_PATH), "_ZN3hmc8mp8_tileEiPi")   # hmc::mp8_tile(int, int32_t*)
    f.argtypes, f.restype = [C.c_int, C.POINTER(C.c_int32)], None
    t = (C.c_int32 * 3)()
    f(K, t)
    return tuple(t)


@pytest.mark.parametrize("K,depth", [(64, 1), (96, 3), (128, 3), (144, 4), (160, 5), (176, 7), (200, 7), (224, 9), (240, 10),
                                     (250, 13), (256, 15), (280, 18), (300, 6), (320, 27)])
def test_depth(K, depth):
    assert tile(K)[2] == depth


def test_every_edge_fits_a_block():
    for K in range(4, 1026, 2):
        x, y, z = tile(K)
        assert 1 <= min(x, y, z) and max(x, y, z) <= K // 2 and (x + 1) * (y + 1) <= 256, K
