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


# all pairs of at most 16 queries on a digit database: (N, limbs, d, chunks, queries,
# time of the vector schedule, of the matrix-core schedule) of whole calls, in us
SMALL_BATCH = [
    (8192, 3, 96, 128, 2, 629, 757), (8192, 3, 128, 128, 2, 809, 896),
    (8192, 3, 64, 128, 2, 542, 570), (4096, 2, 96, 128, 2, 249, 281),
    (8192, 3, 96, 123, 8, 1309, 1161), (8192, 3, 64, 123, 6, 907, 813),
    (8192, 3, 128, 140, 5, 1628, 1296), (8192, 3, 128, 37, 15, 1304, 1202),
    (8192, 3, 96, 64, 9, 1036, 897), (4096, 2, 128, 64, 9, 411, 358),
    (4096, 2, 96, 200, 12, 1043, 819), (16384, 4, 96, 60, 16, 3809, 3667),
    (2048, 1, 64, 300, 5, 200, 155), (2048, 1, 64, 100, 5, 88, 77),
    (2048, 1, 64, 64, 6, 65, 72), (2048, 1, 64, 64, 9, 83, 86),
    (256, 1, 96, 64, 5, 48, 69), (256, 1, 96, 64, 16, 56, 75), (256, 1, 96, 300, 6, 69, 79),
    (256, 1, 96, 300, 12, 84, 91), (256, 1, 96, 300, 15, 103, 99)]


@pytest.mark.parametrize("N,L,d,C,Q,vector,matrix", SMALL_BATCH)
def test_small_batch_schedule(lib, N, L, d, C, Q, vector, matrix):
    # bool mfma_expected_faster(Q, C, d, N, L, small)
    f = lib["_ZN5sanns20mfma_expected_fasterEjjjjjb"]
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.c_uint] * 5 + [ctypes.c_bool]
    assert f(Q, C, d, N, L, True) == (matrix < vector)
