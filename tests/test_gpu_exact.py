"""The short quotients and roots of pvq_exact_dev.h have the bits of the division and the square root: over every float of their
range, every integer and significand, or, for quotients of two floats, many samples and the hardest ones."""
import pytest

import paper_2410_16926_amd as pvq

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

FROM, TO = (127 - 100) << 23, (127 + 100) << 23      # bits of 2^-100 and 2^100


def one_exponent(e):
    return (127 + e) << 23, 1 << 23


def test_reciprocals_and_roots_of_every_float():
    assert pvq.pvq_exact_selftest("reciprocal", FROM, TO - FROM) == 0
    assert pvq.pvq_exact_selftest("root", FROM, TO - FROM) == 0


@pytest.mark.parametrize("exponent", [-100, 0, 99])
def test_integers_over_every_significand(exponent):
    # (a power of two moves divisor, reciprocal and quotient alike while none of them leaves the type's normal range)
    assert pvq.pvq_exact_selftest("small_over", *one_exponent(exponent), ks=range(1, 256)) == 0
    assert pvq.pvq_exact_selftest("integer_over", *one_exponent(exponent), ks=range(1, 1024)) == 0


def test_roots_of_integers_as_divisors():
    assert pvq.pvq_exact_selftest("root_divisor", 1, 65536) == 0


def test_quotients():
    assert pvq.pvq_exact_selftest("divide", 0, 1 << 32, ks=(1, 2, 3)) == 0


def test_what_is_out_of_range_is_refused():
    for what, first, count, k in (("root", FROM - 1, 2, 0), ("root", TO, 1, 0), ("small_over", FROM, 1, 0), ("small_over", FROM, 1, 256),
                                  ("integer_over", FROM, 1, 1024), ("root_divisor", 0, 1, 0), ("root_divisor", 65536, 2, 0)):
        with pytest.raises(pvq.PvqError) as e:
            pvq.pvq_exact_selftest(what, first, count, ks=(k,))
        assert e.value.status == -1
