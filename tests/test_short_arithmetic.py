"""The short root and division of the update pass against correctly rounded ones: every input that can go wrong."""
import ctypes as C

import pytest

import short_arithmetic_build
from conftest import say


@pytest.fixture(scope="module")
def lib():
    return C.CDLL(short_arithmetic_build.build())


def test_quotients_next_to_a_rounding_boundary(lib):
    """For every divisor the dividends whose quotient lies within 32 / (2 D) ulp of a boundary between two roundings (the last
    intermediate is off by 2^-22 ulp at most, that is by less than 8 / (2 D)): all correct with the nearest reciprocal
    estimate, and with one that is an ulp off for all divisors but two, for which v_rcp_f32 returns the nearest (below)."""
    out, divisors = (C.c_int64 * 3)(), (C.c_uint32 * 64)()
    assert lib.quotients(0, 1, out, divisors) == 0
    assert list(out) == [186070940, 0, 3]
    assert set(divisors[:3]) == {0x3FFFFFFF, 0x3FFFFFFD}


@pytest.mark.gpu
@pytest.mark.parametrize("exponent", [27, 28, 47, 67, 90, 107, 126, 127, 150, 186])
def test_every_root_and_reciprocal_of_two_binades(lib, exponent):
    """Over the range of exponents in which the update takes them: the root of every significand and parity, the reciprocal
    estimate of every significand within an ulp, and the nearest for the two divisors that need it."""
    out = (C.c_int64 * 6)()
    say(f"short roots and reciprocals from 2^{exponent - 127}")
    assert lib.roots_and_reciprocals(exponent, out) == 0
    assert list(out) == [0, 0, 0, 0, 0, 0]
