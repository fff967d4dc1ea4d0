"""The exponentials of csrc/math64.h, compiled for the host, against extended
precision.  Bound: 1.5 ulp (the reduced argument and the last two steps round)."""
import ctypes
import math
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#define M64_FN static inline
#include <cmath>
#include "math64.h"
extern "C" void run(int f, const double* a, double* o, double* p, long n) {
  for (long i = 0; i < n; ++i) switch (f) {
    case 1: o[i] = m64::fexp(a[i]); break;
    case 2: o[i] = m64::fexp_neg(a[i]); break;
  }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("m64e")
    (d / "m.cpp").write_text(SRC)
    subprocess.run(["g++", "-O1", "-std=gnu++17", "-ffp-contract=off", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2108_03409_amd", "csrc"), str(d / "m.cpp"), "-o", str(d / "m.so")],
                   check=True)
    L = ctypes.CDLL(str(d / "m.so"))

    def run(f, a):
        a = np.ascontiguousarray(a, dtype=np.float64)
        o, p = np.zeros_like(a), np.zeros_like(a)
        P = ctypes.POINTER(ctypes.c_double)
        L.run(f, *(x.ctypes.data_as(P) for x in (a, o, p)), ctypes.c_long(a.size))
        return (o, p) if f == 0 else o
    return run


def _ulps(got, ref):
    return np.abs(got.astype(np.longdouble) - ref) / np.spacing(np.abs(ref.astype(np.float64)))


def test_exponentials(lib):
    rng = np.random.default_rng(1)
    u = rng.uniform(-1, 1, 200000)
    x = np.concatenate([u * 700, u, 1e-3 * u, 1e-18 * u, np.arange(-1022, 1024) * math.log(2.0)])
    x = x[(x > -708) & (x < 709.7)]
    assert _ulps(lib(1, x), np.exp(x.astype(np.longdouble))).max() <= 1.5
    ref = np.exp(-np.abs(x.astype(np.longdouble)))
    ok = np.abs(x) < 708
    assert _ulps(lib(2, x), ref)[ok].max() <= 1.5
    sub = np.linspace(-745, -708.5, 1000)  # subnormal results: one more rounding, of the smallest unit
    assert _ulps(lib(1, sub), np.exp(sub.astype(np.longdouble))).max() <= 2.5
    assert np.array_equal(lib(2, sub), lib(1, sub)) and np.array_equal(lib(2, -sub), lib(1, sub))


def test_exponential_special_values(lib):
    sp = np.array([0.0, -0.0, np.inf, -np.inf, np.nan, 800.0, -800.0, 1e5, -1e5, 1e308, -1e308, 709.9, -746.0])
    with np.errstate(all="ignore"):
        assert np.array_equal(lib(1, sp), np.exp(sp), equal_nan=True)
        assert np.array_equal(lib(2, sp), np.exp(-np.abs(sp)), equal_nan=True)
