"""Host check of exp_of_logit (csrc/spec_accept.hip) with the split of 256 / (T ln2) that the library makes (csrc/temp_scale.hpp), and with a
shift: the same steps on exact rationals."""
from decimal import Decimal
from fractions import Fraction
import math

import numpy as np
import pytest

from test_exp_of_logit import LN2, constants, fma
from test_exp_table import table
from test_temp_scale import scale_of  # noqa: F401 (temp_scale.hpp itself)


def exp_of_logit(z, scale, k, tab, shift=0):
    """exp(z / T) / 2^shift."""
    c, hi, lo, _ = scale
    magic = k["magic"] - 256.0 * shift
    t = fma(z, c, magic)
    n = t - magic
    assert Fraction(fma(z, hi, -n)) == Fraction(z) * Fraction(hi) - Fraction(n)  # exact: 24 bits times 29
    r = fma(z, lo, fma(z, hi, -n))
    s = fma(fma(fma(fma(k["a4"], r, k["a3"]), r, k["a2"]), r, k["a1"]), r, 1.0)
    low = int(t - k["magic"])  # n less 256 shift: the low word
    assert abs(low) < 2 ** 31
    return math.ldexp(tab[low & 255], low >> 8) * s


@pytest.mark.parametrize("T", [1.0, 0.7, 0.3, 0.05, 1.8])
def test_as_the_library_splits(T, scale_of):
    k, tab, scale = constants(), table(), scale_of(T)
    rng = np.random.default_rng(9)
    zs = np.concatenate([rng.normal(0, 2, 300), rng.uniform(-600 * T, 600 * T, 100), [0.0, 600 * T, -600 * T]]).astype(np.float32)
    # the table's value and the series' last addition 1.1e-16 each, their product as much again
    for z in zs:
        z = float(z)
        want = (Decimal(z) / Decimal(T)).exp()
        assert abs(Decimal(exp_of_logit(z, scale, k, tab)) / want - 1) < Decimal("3.4e-16")


@pytest.mark.parametrize("T", [1.0, 0.7, 0.004, 1e-8])
@pytest.mark.parametrize("units", [900.0, -1700.0, 3e6, -2e9, 4.9e12])
def test_shifted(T, units, scale_of):
    """Logits around `units` temperatures, each against the exact quotient of the float that it is."""
    k, tab, scale = constants(), table(), scale_of(T)
    shift = float(round(Decimal(float(np.float32(units * T))) / Decimal(T) / LN2))  # by a logit, as the kernels take it
    rng = np.random.default_rng(3)
    zs = np.concatenate([(units + rng.uniform(-690, 600, 200)) * T, [units * T]]).astype(np.float32)
    tested = 0
    for z in map(float, zs):
        x = Decimal(z) / Decimal(T) - Decimal(shift) * LN2
        if not -690 < x < 600:  # (floats of a large size lie further apart)
            continue
        tested += 1
        got = Decimal(exp_of_logit(z, scale, k, tab, shift))
        # c_hi + c_lo is good to 2^-62 of itself, and so is their part of the argument
        assert abs(got / x.exp() - 1) < Decimal("3.4e-16") + abs(Decimal(units)) * Decimal(2) ** -61
    assert tested > (100 if abs(units) < 1e9 else 0)
