"""The short root and division of the update pass against correctly rounded ones: every input that can go wrong."""
import ctypes as C

import numpy as np
import pytest

import short_arithmetic_build
import tame_cases
from conftest import say
from paper_2310_18313_amd import binding as B


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


def test_cases_around_the_ends_of_the_range_reach_every_end(lib):
    """The tensors that the GPU test of the update's ends steps: which of them take the short arithmetic, by the library's own
    rule; of the others, every condition of the rule is the only one that some tensor misses, those apart that cannot be."""
    alone, counts = set(), {}
    for name, kw in tame_cases.HPS.items():
        for master in (B.STATE_F16, B.STATE_F32):
            const = tame_cases.host_constants(B.adam_hparams(**kw))
            s = tame_cases.scales(name, master)
            hp, short = (C.c_float * 7)(*const[:7]), 0
            for t in range(tame_cases.N_TENSORS):
                inv = [np.float32(1.0) / s[k][t] for k in ("g_meta", "m_meta", "v_meta", "w_meta")]
                out = tame_cases.missed(const, inv)
                assert bool(lib.tame(hp, (C.c_float * 4)(*inv), C.c_float(const[7]))) == (not out), (name, master, t, out)
                short += not out
                if len(out) == 1:
                    alone |= out
            counts[name, master] = short
    assert alone == tame_cases.CONDITIONS
    for (name, _), short in counts.items():
        if name in ("small beta1", "small beta2"):
            assert short == 0
        elif name == "huge eps":
            assert 0 < short < 50
        else:
            assert 200 < short < 500, (name, short)


@pytest.mark.gpu
@pytest.mark.parametrize("exponent", [27, 28, 47, 67, 90, 107, 126, 127, 150, 186])
def test_every_root_and_reciprocal_of_two_binades(lib, exponent):
    """Over the range of exponents in which the update takes them: the root of every significand and parity, the reciprocal
    estimate of every significand within an ulp, and the nearest for the two divisors that need it."""
    out = (C.c_int64 * 6)()
    say(f"short roots and reciprocals from 2^{exponent - 127}")
    assert lib.roots_and_reciprocals(exponent, out) == 0
    assert list(out) == [0, 0, 0, 0, 0, 0]
