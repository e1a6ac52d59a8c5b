"""The launch rules of the native library on the host, without a device: a rule
that chooses between two kernels has to choose the one that measured faster."""
import ctypes

import pytest

from paper_1904_02033_amd import native as nat


@pytest.fixture(scope="module")
def lib():
    return nat.load()


# one query against few chunks: (log2 N, limbs, d, chunks, time of the split form,
# time of the 1 x 8 tiles) of whole calls, in us
SPLIT = [
    (13, 3, 96, 2, 71, 119), (13, 3, 96, 12, 100, 130), (13, 3, 96, 20, 156, 167),
    (13, 3, 96, 28, 194, 186), (13, 3, 96, 32, 218, 194), (13, 3, 96, 40, 252, 214),
    (13, 3, 128, 12, 139, 153), (13, 3, 128, 14, 169, 159), (13, 3, 128, 16, 179, 163),
    (13, 3, 128, 40, 305, 263), (13, 3, 50, 24, 100, 116), (13, 3, 16, 2, 41, 49),
    (13, 3, 16, 12, 61, 57), (13, 3, 16, 40, 90, 79), (13, 3, 784, 12, 597, 767),
    (13, 3, 200, 12, 198, 220), (13, 2, 128, 20, 146, 152), (13, 2, 128, 24, 173, 159),
    (13, 1, 96, 30, 80, 116), (13, 1, 96, 60, 144, 135), (14, 4, 128, 1, 142, 188),
    (14, 4, 128, 5, 245, 205), (14, 4, 128, 8, 271, 221), (14, 2, 96, 8, 112, 142),
    (12, 2, 128, 40, 107, 125), (12, 2, 128, 56, 135, 139), (12, 2, 32, 80, 64, 70),
    (12, 2, 128, 90, 208, 194), (12, 2, 32, 40, 47, 51),
    (12, 2, 32, 120, 85, 77), (11, 1, 64, 240, 71, 78), (11, 1, 64, 480, 143, 118),
    (10, 1, 64, 400, 64, 75), (10, 1, 64, 1000, 149, 116), (8, 1, 64, 1792, 65, 77)]


@pytest.mark.parametrize("logn,L,d,C,split,tiles", SPLIT)
def test_one_query_form(lib, logn, L, d, C, split, tiles):
    f = lib["_ZN5sanns14mac_split_tileEiiii"]  # int mac_split_tile(logN, C, L, d)
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_int] * 4
    assert (f(logn, C, L, d) > 0) == (split < tiles)
