"""Host check of csrc/temp_scale.hpp, compiled as it is: what the kernels take for a temperature, from the smallest to the largest
that a call may have."""
import ctypes
import os
import subprocess
from decimal import Decimal, getcontext

import numpy as np
import pytest

from test_exp_table import CSRC

getcontext().prec = 50
SOURCE = """
#include "temp_scale.hpp"
extern "C" void scale_of(double T, double* out) {
    const fsr::TempScale t = fsr::temp_scale(T);
    out[0] = t.c; out[1] = t.c_hi; out[2] = t.c_lo; out[3] = t.reach;
}
"""


@pytest.fixture(scope="module")
def scale_of(tmp_path_factory):
    d = tmp_path_factory.mktemp("temp_scale")
    src, lib = d / "scale.cpp", d / "scale.so"
    src.write_text(SOURCE)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-I", CSRC, str(src), "-o", str(lib)])
    f = ctypes.CDLL(str(lib)).scale_of
    f.argtypes = [ctypes.c_double, ctypes.POINTER(ctypes.c_double)]

    def call(T):
        out = (ctypes.c_double * 4)()
        f(T, out)
        return list(out)
    return call


@pytest.mark.parametrize("T", [1.0, 0.7, 0.3, 0.05, 1.8, 1e-30, 2.1e-41, 1e30, 5e35])
def test_parts(scale_of, T):
    c, hi, lo, reach = scale_of(T)
    exact = Decimal(256) / (Decimal(2).ln() * Decimal(T))
    assert c == float(exact)
    assert hi != 0 and int(np.frexp(hi)[0] * 2.0 ** 29) == np.frexp(hi)[0] * 2.0 ** 29  # 29 bits: times a logit's 24 exact
    # the rest is rounded from long double's 64 bits, 2^-63 of the whole
    assert abs(Decimal(hi) + Decimal(lo) - exact) <= exact * Decimal(2) ** -62
    assert reach > 0


@pytest.mark.parametrize("T", [5e-324, 1e-310, 1e-300, 1e-60, 1e-50, 1e-48, 1e-45, 1e-44, 1e-42, 1.9e-41, 2.1e-41, 1e-38, 1e-20, 1e-3, 1.0, 1e3,
                               1e30, 5e35, 6e35, 1e36, 1e37, 1e38, 3e38, 1e45, 1e300, 1.7e308])
def test_a_logit_at_the_reach_is_600_temperatures(scale_of, T):
    """Masked logits count as -reach, which adds nothing only if that is -600 temperatures."""
    reach = scale_of(T)[3]
    assert reach == -1.0 or abs(reach / T / 600.0 - 1.0) < 2.0 ** -23
