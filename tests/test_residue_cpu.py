"""Residue arithmetic and dispatch of the INT8 projector products (host arithmetic)."""
import ctypes

import pytest

from paper_1406_4350_amd import chebfd as cf


def _limits(l, x0=0, x1=0):
    v = [ctypes.c_int() for _ in range(6)]
    st = cf.load_library().cheb_residue_limits(l, x0, x1, *[ctypes.byref(x) for x in v])
    return (st, *[x.value for x in v])


def test_residues_of_every_integer_of_the_split_stay_within_the_accumulator_bound():
    """Every integer that the split of an operand may reduce, for every modulus: the largest residue left is within the
    one that the int32 accumulators of the longest product are sized by."""
    _, count, *_ = _limits(0)
    for l in range(count):
        st, _, p, top, bound, max_k, _ = _limits(l)
        assert st == cf.CHEB_OK
        *_, largest = _limits(l, -top, top + 1)
        assert (p - 1) // 2 <= largest <= bound, (p, largest, bound)
        if p % 2:
            assert bound * bound * max_k < 2 ** 31
            assert bound <= 127


def test_limits_arguments():
    _, count, *_ = _limits(0)
    assert _limits(-1)[0] == _limits(count)[0] == _limits(0, 2, 1)[0] == cf.CHEB_ERR_ARG
    assert cf.load_library().cheb_residue_limits(0, 0, 0, *[None] * 6) == cf.CHEB_ERR_ARG


# (M, N, K, measured us on the FP64 and on the INT8 matrix cores); M > K: P w
MEASURED = [
    (3328, 512, 137065, 21987, 10833),
    (137065, 512, 3328, 21828, 12210),
    (3328, 128, 137065, 9352, 5964),
    (137065, 128, 3328, 5651, 5956),
    (3328, 64, 137065, 5722, 5587),
    (137065, 64, 3328, 3229, 5512),
    (1664, 700, 57777, 6285, 3912),
    (57777, 700, 1664, 6580, 4508),
    (832, 512, 57777, 3733, 1920),
    (57777, 512, 832, 2639, 2331),
    (512, 448, 17077, 639, 383),
    (17077, 448, 512, 502, 545),
    (512, 512, 17077, 417, 398),
    (17077, 512, 512, 563, 586),
    (512, 256, 17077, 213, 291),
    (17077, 256, 512, 310, 307),
    (1024, 512, 7153, 348, 273),
    (7153, 512, 1024, 438, 329),
    (832, 320, 17077, 797, 510),
    (17077, 320, 832, 557, 587),
    (3328, 96, 137065, 9266, 5767),
    (137065, 96, 3328, 5770, 5744),
    (256, 1024, 57777, 1378, 1756),
    (57777, 1024, 256, 2123, 3377),
    (57777, 1024, 512, 3464, 3863),
    (832, 128, 33401, 628, 512),
    (33401, 128, 832, 465, 574),
    (256, 256, 7153, 53, 109),
    (7153, 256, 256, 71, 112)]


@pytest.mark.parametrize("M,N,K,fp64,int8", MEASURED)
def test_route_is_the_faster_side_of_the_measured_shapes(M, N, K, fp64, int8):
    """The side taken is the faster one, or one within 5% of it (runs of one side differ by some 2%)."""
    v, a, b = ctypes.c_int(), ctypes.c_double(), ctypes.c_double()
    assert cf.load_library().cheb_product_route(M, N, K, int(M > K), ctypes.byref(v), ctypes.byref(a),
                                                ctypes.byref(b)) == cf.CHEB_OK
    assert (int8 if v.value else fp64) <= 1.05 * min(fp64, int8), (a.value, b.value)
    assert 0.8 < a.value / fp64 < 1.25 and 0.8 < b.value / int8 < 1.25


def test_small_products_keep_the_small_gemm():
    """Products of K <= 1024 and at most 1024 blocks of 16 x 16 have one FP64 kernel without another route."""
    v, a, b = ctypes.c_int(), ctypes.c_double(), ctypes.c_double()
    for back in (0, 1):
        for M in range(16, 4097, 240):
            for K in range(64, 1025, 96):
                N = 16 * (1024 // ((M + 15) // 16))
                assert cf.load_library().cheb_product_route(M, N, K, back, ctypes.byref(v), ctypes.byref(a),
                                                            ctypes.byref(b)) == cf.CHEB_OK and v.value == 0, (M, N, K)


def test_route_arguments_and_longest_product():
    lib = cf.load_library()
    v, a, b = ctypes.c_int(), ctypes.c_double(), ctypes.c_double()
    ref = ctypes.byref(v), ctypes.byref(a), ctypes.byref(b)
    _, _, _, _, _, max_k, _ = _limits(0)
    assert lib.cheb_product_route(1664, 512, max_k, 0, *ref) == cf.CHEB_OK and v.value == 1
    assert lib.cheb_product_route(1664, 512, max_k + 1, 0, *ref) == cf.CHEB_OK and v.value == 0
    for M, N, K in ((0, 512, 9000), (512, 0, 9000), (512, 512, 0)):
        assert lib.cheb_product_route(M, N, K, 0, *ref) == cf.CHEB_OK and v.value == 0
    assert lib.cheb_product_route(1, 1, 1, 0, None, ref[1], ref[2]) == cf.CHEB_ERR_ARG
