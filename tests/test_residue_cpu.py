"""Residue arithmetic of the INT8 projector products (host arithmetic, the operations of the kernels)."""
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
