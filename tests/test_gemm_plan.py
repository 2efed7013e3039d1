"""The tile shape and K split that a backbone GEMM's size gets, asked on the CPU."""
import ctypes as C
import random

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


@pytest.mark.parametrize("n,rows", [(4096, 1), (4096, 33), (4096, 64), (4096, 128), (2048, 1), (2048, 64)])
def test_ranges_do_not_start_on_the_same_channels(lib, n, rows):
    """K = 16,384: ranges that start whole multiples of 4 KB apart take a fifth longer
    (one row, 4,096 columns, four and eight ranges 34 and 37 us, three to six 30 to 32)."""
    s = gemm_plan(lib, RESID, rows, n, 16384)[2]
    assert s > 1 and 16384 % (2048 * s) != 0


@pytest.mark.parametrize("rows", [107, 128])
def test_no_split_where_one_range_is_bound_by_its_weights(lib, rows):
    """16,384 x 4,096 at 128 rows: 37 us in one launch, 36 and a reduction of 5 in two ranges."""
    assert gemm_plan(lib, GELU, rows, 16384, 4096)[2] == 1


def test_launches_fit_a_dispatch(lib):
    """The largest batches that the backbone accepts (rows x columns / 32 below 2^32):
    no launch of the plan holds 2^32 work-items of its 256 threads a tile."""
    rng = random.Random(3)
    for _ in range(400):
        d = 128 * rng.randint(1, 32)
        f = 128 * int(2 ** rng.uniform(0, 15))
        glu = rng.random() < 0.5
        widest = max(3 * d, (1 + glu) * f)
        rows = ((1 << 32) - 1) // 512 // -(-widest // 128) * 128
        rows = min(int(rows * rng.choice((1.0, 1.0, rng.random()))), (1 << 31) - 2)
        for epi, n, k in ((BF16, 3 * d, d), (RESID, d, d), (GEGLU if glu else GELU, f, d), (RESID, d, f)):
            m1, shape, ranges = gemm_plan(lib, epi, rows, n, k)
            columns = n * (2 if epi == GEGLU else 1)
            for m, s, r in ((m1, "256x256", 1), (rows - m1, shape, ranges)):
                bn, bm = map(int, s.split("x"))
                assert -(-m // bm) * -(-columns // bn) * r * 256 < 1 << 32, (rows, n, k, s, r)
