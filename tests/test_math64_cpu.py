"""The float64 elementary functions of csrc/math64.h, compiled for the host,
against extended precision.  Bounds: the reduced polynomials err below 2e-17 of
the result, each function adds at most a few roundings of its last steps:
2 ulp for log, 3 ulp for log1p and atan2, 1.5 units of 2^-53 absolute for sine
and cosine (the two-part reduction errs below 1e5 2^-110)."""
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
extern "C" void run(int f, const double* a, const double* b, double* o, double* p, long n) {
  for (long i = 0; i < n; ++i) switch (f) {
    case 0: m64::fsincos(a[i], o + i, p + i); break;
    case 1: o[i] = m64::flog(a[i]); break;
    case 2: o[i] = m64::flog1p(a[i]); break;
    case 3: o[i] = m64::fatan2(a[i], b[i]); break;
    case 4: o[i] = m64::wrap_2pi(a[i]); break;
    case 5: o[i] = m64::fdiv(a[i], b[i]); break;
  }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("m64")
    (d / "m.cpp").write_text(SRC)
    subprocess.run(["g++", "-O1", "-std=gnu++17", "-ffp-contract=off", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2108_03409_amd", "csrc"), str(d / "m.cpp"), "-o", str(d / "m.so")],
                   check=True)
    L = ctypes.CDLL(str(d / "m.so"))

    def run(f, a, b=None):
        a = np.ascontiguousarray(a, dtype=np.float64)
        b = a if b is None else np.ascontiguousarray(b, dtype=np.float64)
        o, p = np.empty_like(a), np.empty_like(a)
        P = ctypes.POINTER(ctypes.c_double)
        L.run(f, *(x.ctypes.data_as(P) for x in (a, b, o, p)), ctypes.c_long(a.size))
        return (o, p) if f == 0 else o
    return run


def _ulps(got, ref):
    return np.max(np.abs(got.astype(np.longdouble) - ref) / np.spacing(np.abs(ref.astype(np.float64))))


def test_accuracy(lib):
    rng = np.random.default_rng(0)
    n = 200000
    u = rng.uniform(-1, 1, n)
    for scale in (1e-3, 1.0, 20.0, 1.1e5, 1e9):
        x = u * scale
        s, c = lib(0, x)
        xl = x.astype(np.longdouble)
        for got, ref in ((s, np.sin(xl)), (c, np.cos(xl))):
            assert np.max(np.abs(got.astype(np.longdouble) - ref)) <= 1.5 * 2.0 ** -53
    x = np.concatenate([np.exp(u * 700), 1 + 0.5 * u, rng.uniform(0, 4, n)])
    x = x[(x > 0) & (x != 1)]
    assert _ulps(lib(1, x), np.log(x.astype(np.longdouble))) <= 2
    t = np.concatenate([rng.uniform(-0.999, 3, n), 1e-3 * u, 10.0 ** (-20 * rng.uniform(size=n)) * u, 1e10 * abs(u)])
    t = t[t != 0]
    assert _ulps(lib(2, t), np.log1p(t.astype(np.longdouble))) <= 3
    y, z = u * 10.0 ** (40 * rng.uniform(-0.5, 0.5, n)), rng.uniform(-1, 1, n)
    assert _ulps(lib(3, y, z), np.arctan2(y.astype(np.longdouble), z.astype(np.longdouble))) <= 3
    w = u * 1e3
    assert np.array_equal(lib(4, w), np.array([math.remainder(v, 6.283185307179586477)
                                               for v in w]))
    assert _ulps(lib(5, y, z), y.astype(np.longdouble) / z.astype(np.longdouble)) <= 1


def test_special_values(lib):
    sp = np.array([0.0, -0.0, 1.0, -1.0, np.inf, -np.inf, np.nan, 5e-324, 1e-310, 1e308, -1e308])
    with np.errstate(all="ignore"):
        for f, ref in ((1, np.log), (2, np.log1p)):
            np.testing.assert_allclose(lib(f, sp), ref(sp), rtol=1e-15)
        s, c = lib(0, sp)
        np.testing.assert_allclose(s, np.sin(sp), rtol=1e-15)
        np.testing.assert_allclose(c, np.cos(sp), rtol=1e-15)
        y, x = (g.ravel() for g in np.meshgrid(sp, sp))
        got, ref = lib(3, y, x), np.arctan2(y, x)
        np.testing.assert_allclose(got, ref, rtol=1e-15)
        ok = ~np.isnan(ref)
        assert np.array_equal(np.signbit(got[ok]), np.signbit(ref[ok]))
