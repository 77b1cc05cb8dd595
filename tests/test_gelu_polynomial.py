"""The polynomial behind GELU (csrc/gelu_poly.h), compiled by the host compiler and evaluated in fp32 in the kernel's order,
against the library's erfc in double precision: the errors that its comment states."""

import ctypes as C
import os
import subprocess

import numpy as np
import pytest
from scipy.special import erfc

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_23431_amd", "csrc")

SOURCE = r"""
#include <math.h>
#include "gelu_poly.h"
extern "C" void evaluate(const float *t, float *gelu, double *tail, int n) {
  for (int k = 0; k < n; ++k) {
    const float b = fabsf(t[k]), a = b > 8.f ? 8.f : b;
    float r = gelu_coefficient(GELU_TERMS - 1);
    double q = r;
    for (int i = GELU_TERMS - 2; i >= 0; --i) { r = fmaf(r, a, gelu_coefficient(i)); q = q * a + gelu_coefficient(i); }
    gelu[k] = fmaf(-0.5f * a, exp2f(-(r * a)), t[k] > 0.f ? t[k] : 0.f);
    tail[k] = 0.5 * exp2(-(q * a));          // the coefficients alone
  }
}
"""


@pytest.fixture(scope="module")
def evaluate(tmp_path_factory):
    d = tmp_path_factory.mktemp("gelu")
    (d / "gelu.cpp").write_text(SOURCE)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-mfma", "-ffp-contract=off", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                           str(d / "gelu.cpp"), "-o", str(d / "gelu.so")])
    lib = C.CDLL(str(d / "gelu.so"))

    def call(t):
        t = np.ascontiguousarray(t, np.float32)
        gelu, tail = np.empty_like(t), np.empty(t.shape, np.float64)
        lib.evaluate(t.ctypes.data_as(C.c_void_p), gelu.ctypes.data_as(C.c_void_p), tail.ctypes.data_as(C.c_void_p), t.size)
        return gelu, tail
    return call


def exact(t):
    return t.astype(np.float64) * 0.5 * erfc(-t.astype(np.float64) / np.sqrt(2))


def test_errors_of_the_coefficients(evaluate):
    a = np.linspace(0, 8, 400001).astype(np.float32)
    phi = 0.5 * erfc(a.astype(np.float64) / np.sqrt(2))
    tail = evaluate(a)[1]
    assert np.abs(a * (tail - phi)).max() < 3.2e-9
    for at, relative in ((5, 1.1e-4), (6, 8e-3), (7, 0.11)):
        assert np.abs(tail / phi - 1)[a <= at].max() < relative


def test_errors_in_fp32(evaluate):
    t = np.linspace(-12, 12, 600001).astype(np.float32)
    y, ref = evaluate(t)[0].astype(np.float64), exact(t)
    assert np.abs(y - ref)[t <= 0].max() < 3.4e-8                                  # the whole negative side
    near = (t < 0) & (t >= -3)
    assert (np.abs(y - ref) / np.abs(ref))[near].max() < 9e-7
    assert (np.abs(y - ref) / ref)[t > 0].max() < 1.2e-7                           # an fp32 rounding or two
    rng = np.random.default_rng(7)
    for deviation, bound in ((0.1, 3.2e-8), (1.0, 2.8e-8), (4.0, 1.8e-8)):
        x = (deviation * rng.standard_normal(400000)).astype(np.float32)
        assert np.linalg.norm(evaluate(x)[0] - exact(x)) < bound * np.linalg.norm(exact(x))


def test_ends(evaluate):
    y = evaluate([np.nan, np.inf, 3e38, 0.0, -0.0, -np.inf, -3e38, 9.0, -9.0])[0]
    assert np.isnan(y[0]) and np.isinf(y[1]) and y[2] == np.float32(3e38) and y[3] == 0 and y[4] == 0
    assert (np.abs(y[5:7]) < 1e-14).all() and y[7] == 9 and abs(y[8]) < 1e-14
