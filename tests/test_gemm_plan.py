"""The tile shape and K split that a backbone GEMM's size gets, asked on the CPU."""
import ctypes as C

import pytest

BF16, GELU, RESID, GEGLU = 0, 1, 2, 3
SHAPES = ["256x256", "256x160", "256x128", "128x160", "128x96", "64x96", "128x128"]  # weight rows x tokens


class Plan(C.Structure):
    _fields_ = [("m1", C.c_int32), ("shape", C.c_int32), ("S", C.c_int32)]


def gemm_plan(lib, epi, m, n, k):
    """(rows of a leading launch of 256x256 tiles, shape of the others, K ranges)"""
    f = C.CDLL(lib.lib_path())._ZN3jnx9gemm_planEiiii
    f.restype, f.argtypes = Plan, [C.c_int, C.c_int32, C.c_int32, C.c_int32]
    p = f(epi, m, n, k)
    return p.m1, SHAPES[p.shape], p.S


@pytest.mark.parametrize("rows", [1, 33, 64])
def test_ranges_no_faster_than_the_weights_arrive(lib, rows):
    """134 MB of weights take 28 to 31 us however many ranges are fetched at once (one
    row in three ranges 32 us, in eight, 256 workgroups, 37)."""
    assert gemm_plan(lib, RESID, rows, 4096, 16384)[2] <= 6


@pytest.mark.parametrize("rows", [107, 128])
def test_no_split_where_one_range_is_bound_by_its_weights(lib, rows):
    """16,384 x 4,096 at 128 rows: 37 us in one launch, 36 and a reduction of 5 in two ranges."""
    assert gemm_plan(lib, GELU, rows, 16384, 4096)[2] == 1
