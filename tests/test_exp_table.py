"""Host check of the table behind exp_lookup (csrc/spec_accept.hip): the kernel's constants and exp_table.inc, put through
the same steps in numpy, give exp to a few 1e-16, and the table is what its generator prints."""
import importlib.util
import os
import re

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_20503_amd", "csrc")
LD = np.longdouble


def table():
    text = open(os.path.join(CSRC, "exp_table.inc")).read()
    return np.array([float.fromhex(x) for x in re.findall(r"0x[0-9a-f.]+p[+-]\d+", text)])


def constants():
    text = open(os.path.join(CSRC, "spec_accept.hip")).read()
    body = text[text.index("ExpTable exp_table("):]
    body = body[:body.index("return k;")]
    vals = {m.group(1): float(m.group(2)) for m in re.finditer(r"k\.(\w+) = (-?[0-9.e+-]+);", body)}
    vals["floor"] = float(re.search(r"kExpTableFloor = (-[0-9.]+);", text).group(1))
    return vals


def lookup_like_the_kernel(x, k, tab):
    x = np.fmax(x, k["floor"])
    t = x * k["c"] + k["magic"]
    kf = t - k["magic"]
    n = (t.view(np.uint64) & np.uint64(0xFFFFFFFF)).astype(np.uint32)
    bits = tab.view(np.uint64)
    j = n & np.uint32(255)
    hi = (bits >> np.uint64(32)).astype(np.uint32) - (np.arange(256, dtype=np.uint32) << np.uint32(12))
    word = hi[j] + (n << np.uint32(12))
    pow2 = ((word.astype(np.uint64) << np.uint64(32)) | (bits[j] & np.uint64(0xFFFFFFFF))).view(np.float64)
    r = (x + kf * k["nl_hi"]) + kf * k["nl_lo"]
    p = ((r * (1.0 / 24.0) + 1.0 / 6.0) * r + 0.5) * r + 1.0
    return (pow2 * r) * p + pow2


def test_table_and_generator():
    tab = table()
    spec = importlib.util.spec_from_file_location("gen", os.path.join(CSRC, "exp_poly_coefficients.py"))
    gen = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(gen)
    assert len(tab) == 256 and np.array_equal(tab, np.array(gen.table()))
    exact = np.exp2(np.arange(256, dtype=LD) / 256)
    assert float(np.max(np.abs(tab.astype(LD) / exact - 1))) < 1.2e-16  # each value rounded to nearest (half an ulp: 1.1e-16)


@pytest.mark.parametrize("lo,hi", [(-1e-3, 0.0), (-40.0, 0.0), (-700.0, 0.0), (0.0, 120.0)])
def test_lookup_is_exp(lo, hi):
    x = np.random.default_rng(3).uniform(lo, hi, 200000)
    got = lookup_like_the_kernel(x, constants(), table())
    # rounding of the table value, of the product and of the sum: 1.1e-16 + 1e-3 * 2.2e-16 + 1.1e-16; numpy rounds the
    # two steps of r separately, which adds half an ulp of x - n ln2 / 256 <= 1.4e-3 and of x itself where n is large
    assert float(np.max(np.abs(got.astype(LD) / np.exp(x.astype(LD)) - 1))) < 3e-16 + 1.2e-16 * max(1.0, abs(lo), abs(hi))


def test_arguments_past_the_floor():
    got = lookup_like_the_kernel(np.array([0.0, -701.0, -1e6, -np.inf, np.nan]), constants(), table())
    assert got[0] == 1.0 and np.all(got[1:] > 0) and np.all(got[1:] < 1e-303)
