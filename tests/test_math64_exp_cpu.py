"""The exponentials of csrc/math64.h, and its sine, cosine and remainder by 2 pi at
large arguments, compiled for the host, against extended precision (arguments
reduced with integers where that does not reach).  Bounds: exponential 1.5 ulp (the
reduced argument and the last two steps round); sine and cosine 2.5 units of 2^-53
from 1e5 to 2^54, where two of the reduction's sums round near pi / 2, and 1.5 beyond,
where the reduced argument rounds once; the remainder is exact."""
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
    case 0: m64::fsincos(a[i], o + i, p + i); break;
    case 1: o[i] = m64::fexp(a[i]); break;
    case 2: o[i] = m64::fexp_neg(a[i]); break;
    case 3: o[i] = m64::wrap_2pi(a[i]); break;
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


def _pi(bits):
    def atan_inv(n):
        t = s = (1 << bits) // n
        k = 1
        while t:
            t //= n * n
            k += 2
            s += -(t // k) if k // 2 % 2 else t // k
        return s
    return 4 * (4 * atan_inv(5) - atan_inv(239))


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


def test_sine_and_cosine_of_large_arguments(lib):
    rng = np.random.default_rng(2)
    x = np.concatenate([2.0 ** rng.uniform(17, 54, 3000), 2.0 ** rng.uniform(54, 1023.9, 3000),
                        2.0 ** np.arange(17, 1024), [np.finfo(np.float64).max, 6381956970095103.0 * 2.0 ** 797]])
    x *= np.where(rng.random(x.size) < 0.5, -1.0, 1.0)
    s, c = lib(0, x)
    bits, sc = 2400, 64
    two_pi = 2 * _pi(bits)
    for v, sv, cv in zip(x, s, c):
        n, d = v.as_integer_ratio()  # d is a power of two
        r = ((n << bits) // d) % two_pi
        q, r = divmod(r, two_pi // 4)
        # the fraction of the quadrant as the sum of two extended numbers
        h = r >> (bits - sc)
        lo = (r - (h << (bits - sc))) >> (bits - 2 * sc)
        t = np.longdouble(h) / np.longdouble(2 ** sc) + np.longdouble(lo) / np.longdouble(2 ** sc) ** 2
        S, C = np.sin(t), np.cos(t)
        rs, rc = ((S, C), (C, -S), (-S, -C), (-C, S))[q & 3]
        tol = (1.5 if abs(v) >= 2.0 ** 54 else 2.5) * 2.0 ** -53
        assert abs(sv - rs) <= tol and abs(cv - rc) <= tol, v
    with np.errstate(all="ignore"):
        s, c = lib(0, np.array([np.inf, -np.inf, np.nan]))
    assert np.isnan(s).all() and np.isnan(c).all()


def test_remainder_of_large_arguments(lib):
    rng = np.random.default_rng(3)
    y = np.concatenate([2.0 ** rng.uniform(-3, 1023.9, 5000), 2.0 ** np.arange(40, 1024), [np.finfo(np.float64).max]])
    y *= np.where(rng.random(y.size) < 0.5, -1.0, 1.0)
    assert np.array_equal(lib(3, y), np.array([math.remainder(v, 6.283185307179586477) for v in y]))
    with np.errstate(all="ignore"):
        assert np.isnan(lib(3, np.array([np.inf, -np.inf, np.nan]))).all()
