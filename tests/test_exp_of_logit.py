"""Host check of exp_of_logit (csrc/spec_accept.hip): its constants and the split of 256 / (T ln2), put through the same steps,
give exp(z / T) to a few 1e-16 at every temperature, up to the reach that the kernels keep to."""
import os
import re
from decimal import Decimal, getcontext
from fractions import Fraction
import math

import numpy as np
import pytest

from test_exp_table import CSRC, table

getcontext().prec = 50
LN2 = Decimal(2).ln()


def constants():
    text = open(os.path.join(CSRC, "spec_accept.hip")).read()
    body = text[text.index("ExpDirect exp_direct("):]
    body = body[:body.index("return k;")]
    return {m.group(1): float(m.group(2)) for m in re.finditer(r"k\.(\w+) = (-?[0-9.e+-]+);", body)}


def fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))


def exp_of_logit(z, T, k, tab):
    exact = Decimal(256) / (LN2 * Decimal(T))
    c = float(exact)
    m, e = math.frexp(c)
    hi = math.ldexp(math.floor(m * 2.0 ** 29), e - 29)
    lo = float(exact - Decimal(hi))
    n = fma(z, c, k["magic"]) - k["magic"]
    assert fma(z, hi, -n) == float(Fraction(z) * Fraction(hi) - Fraction(n))  # exact: 24 bits times 29
    r = fma(z, lo, fma(z, hi, -n))
    s = fma(fma(fma(fma(k["a4"], r, k["a3"]), r, k["a2"]), r, k["a1"]), r, 1.0)
    return math.ldexp(tab[int(n) & 255], int(n) >> 8) * s


def test_series():
    k = constants()
    for n in range(1, 5):
        assert k[f"a{n}"] == float((LN2 / 256) ** n / math.factorial(n))


@pytest.mark.parametrize("T", [1.0, 0.7, 0.3, 0.05, 1.8])
def test_exp_of_logit_is_exp(T):
    k, tab = constants(), table()
    rng = np.random.default_rng(9)
    zs = np.concatenate([rng.normal(0, 2, 300), rng.uniform(-600 * T, 600 * T, 100), [0.0, 600 * T, -600 * T]]).astype(np.float32)
    # the table's value and the series' last addition 1.1e-16 each, their product as much again
    for z in zs:
        z = float(z)
        want = (Decimal(z) / Decimal(T)).exp()
        assert abs(Decimal(exp_of_logit(z, T, k, tab)) / want - 1) < Decimal("3.4e-16")
