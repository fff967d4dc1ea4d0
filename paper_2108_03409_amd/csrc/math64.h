// Float64 elementary functions for kernels whose time is elementary functions:
// fewer vector instructions than the device library's (exp 27 for 42, sincos 45 for 155, log 43
// for 98, log1p 52 for 135, atan2 64 for 105, remainder by 2 pi 6 for 60), straight-line but for
// sine and cosine from 1e5 and the remainder from 2^30 on.  Polynomials interpolate the reduced
// functions at Chebyshev nodes (approximation error below 2e-17 of the result);
// measured against 113-bit arithmetic over 4 million arguments: exp 1.1 ulp, log 0.9, log1p
// 1.3, atan2 2.2, sine and cosine 1.2e-16 absolute for |x| < 1e5 and from 2^54 on, 1.9e-16
// between; the remainder is exact.  Zeros, infinities and NaN follow the C library.
// What the functions alone gave, in the kernels they came into: log psi of an RBM (N = 64, N_h =
// 256, 16 384 samples, theta included) 88.7 -> 76.8 us, CNN log psi (16 x 16, C = 16, k = 4,
// 1 024 samples) 258 -> 233 us, its local energies (512 samples) 2.15 -> 2.07 ms.  The exact
// reductions of large arguments cost the same CNN's chains 2% (6.41 -> 6.52 ms), its local
// energies 0.6% and log psi 1%.
#pragma once

#include <cmath>

#ifdef __HIP_DEVICE_COMPILE__
#define M64_MANT(x) __builtin_amdgcn_frexp_mant(x)
#define M64_EXPO(x) __builtin_amdgcn_frexp_exp(x)
#define M64_RCP(x) __builtin_amdgcn_rcp(x)
#define M64_MULHI(a, b) __umul64hi(a, b)
#else
inline double m64_mant_host(double x) { int e; return std::frexp(x, &e); }
inline int m64_expo_host(double x) { int e; std::frexp(x, &e); return std::isfinite(x) ? e : 0; }
#define M64_MANT(x) m64_mant_host(x)
#define M64_EXPO(x) m64_expo_host(x)
#define M64_RCP(x) ((double)(1.0f / (float)(x)))
#define M64_MULHI(a, b) ((unsigned long long)(((unsigned __int128)(a) * (b)) >> 64))
#endif
#ifndef M64_FN
#define M64_FN __host__ __device__ __forceinline__
#endif

namespace m64 {

// a b + c for a literal c: the three-operand form with c in scalar registers.  (Left to
// itself the compiler takes the two-operand form, whose accumulator it first fills with the
// literal by two vector moves: three vector instructions instead of one.)
M64_FN double kfma(double a, double b, double c) {
#ifdef __HIP_DEVICE_COMPILE__
  double d;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
  return d;
#else
  return fma(a, b, c);
#endif
}

// a / b for b in the normal range and a quotient that neither over- nor
// underflows: reciprocal refined by two Newton steps, one residual correction
M64_FN double fdiv(double a, double b) {
  double r = M64_RCP(b);
  r = fma(fma(-b, r, 1.0), r, r);
  r = fma(fma(-b, r, 1.0), r, r);
  const double q = a * r;
  return fma(fma(-b, q, a), r, q);
}

// 2^n e^r for x = n ln 2 + r, |r| <= ln 2 / 2
M64_FN double exp_core(double x) {
  const double n = rint(x * 1.4426950408889634);
  double r = fma(n, -0x1.62e42fefa39efp-1, x);
  r = fma(n, -0x1.abc9e3b39803fp-56, r);
  double p = 0x1.af38a9b0ec855p-26;
  p = kfma(p, r, 0x1.289185613a3d6p-22);
  p = kfma(p, r, 0x1.71de0dae63bb3p-19);
  p = kfma(p, r, 0x1.a019b90d2ae7ap-16);
  p = kfma(p, r, 0x1.a01a01a7c41d5p-13);
  p = kfma(p, r, 0x1.6c16c1788bd90p-10);
  p = kfma(p, r, 0x1.11111111109b3p-7);
  p = kfma(p, r, 0x1.5555555553d63p-5);
  p = kfma(p, r, 0x1.5555555555556p-3);
  p = kfma(p, r, 0x1.0000000000001p-1);
  return ldexp(1.0 + fma(r * r, p, r), (int)n);
}
M64_FN double fexp(double x) {
  const double v = exp_core(fmin(fmax(x, -800.0), 800.0));
  return x != x ? x : v;
}
// e^{-|x|}; the first gives 0 for a NaN, for callers that carry x in another term
M64_FN double fexp_neg0(double x) { return exp_core(fmax(-fabs(x), -800.0)); }
M64_FN double fexp_neg(double x) {
  const double v = fexp_neg0(x);
  return x != x ? x : v;
}

// x - n pi/2 and n mod 4 for |x| >= 2^54 (Payne and Hanek's reduction): with |x| = m 2^k, m a
// 53-bit integer, the bits of 2 / pi above weight 2^(1 - k) give multiples of 4 in |x| 2 / pi;
// the product with 192 bits from there on, 128 of its bits kept, is right to 2^-123, and the
// reduced argument, 2^-62 at least, to one rounding.  NaN for an infinite x.
M64_FN double reduce_big(double x, int* q) {
  static constexpr unsigned long long two_over_pi[20] = {
      0xa2f9836e4e441529ull, 0xfc2757d1f534ddc0ull, 0xdb6295993c439041ull, 0xfe5163abdebbc561ull,
      0xb7246e3a424dd2e0ull, 0x06492eea09d1921cull, 0xfe1deb1cb129a73eull, 0xe88235f52ebb4484ull,
      0xe99c7026b45f7e41ull, 0x3991d639835339f4ull, 0x9c845f8bbdf9283bull, 0x1ff897ffde05980full,
      0xef2f118b5a0a6d1full, 0x6d367ecf27cb09b7ull, 0x4f463f669e5fea2dull, 0x7527bac7ebe5f17bull,
      0x3d0739f78a5292eaull, 0x6bfb5fb11f8d5d08ull, 0x56033046fc7b6babull, 0xf0cfbc209af4361dull,
  };
  const int k = M64_EXPO(x) - 53, at = k > 2 ? k - 2 : 0, sh = at & 63;
  const unsigned long long m = (unsigned long long)(fabs(M64_MANT(x)) * 0x1p53);
  const unsigned long long* p = two_over_pi + (at >> 6);
  unsigned long long w[3];
  for (int i = 0; i < 3; ++i) w[i] = sh ? p[i] << sh | p[i + 1] >> (64 - sh) : p[i];
  const unsigned long long c2 = M64_MULHI(m, w[2]), lo = m * w[1] + c2;
  const unsigned long long hi = m * w[0] + M64_MULHI(m, w[1]) + (lo < c2 ? 1 : 0);  // 4 hi.lo / 2^64 = |x| 2 / pi mod 4
  const long long f = (long long)(hi << 2 | lo >> 62);  // the fraction, in [-1/2, 1/2)
  int n = (int)(hi >> 62) + (f < 0 ? 1 : 0);
  const double fh = (double)(f & ~0x7ffll) * 0x1p-64;
  const double fl = fma((double)(lo << 2), 0x1p-128, (double)(f & 0x7ffll) * 0x1p-64);
  double r = fma(fh, 0x1.921fb54442d18p+0, fma(fh, 0x1.1a62633145c07p-54, fl * 0x1.921fb54442d18p+0));
  *q = x < 0.0 ? -n : n;
  r = x < 0.0 ? -r : r;
  return fabs(x) < INFINITY ? r : NAN;
}

// sin and cos of x through r = x - n pi/2, |r| <= pi/4, n = rint(2 x / pi).  x - n P1
// with P1 = fl(pi/2) is exact (both are multiples of 2^-52 and the difference is below
// 2), so the remaining error is that of n (pi/2 - P1).  From 1e5 on the rounding of
// 2 x / pi can be off by an integer, which a second step takes back.
M64_FN void fsincos(double x, double* sp, double* cp) {
  double n = rint(x * 0.63661977236758134);
  double r = fma(n, -0x1.921fb54442d18p+0, x);
  r = fma(n, -0x1.1a62633145c07p-54, r);
  int q = (int)n;
  if (!(fabs(x) < 1e5)) {
    r = fma(n, 0x1.f1976b7ed8fbcp-110, r);
    const double n2 = rint(r * 0.63661977236758134);
    r = fma(n2, -0x1.921fb54442d18p+0, r);
    r = fma(n2, -0x1.1a62633145c07p-54, r);
    q = (int)(n - 4.0 * floor(0.25 * n)) + (int)n2;
    if (!(fabs(x) < 0x1p54)) r = reduce_big(x, &q);
  }
  const double z = r * r;
  double s = 0x1.5e0b05bff20f2p-33;
  s = kfma(s, z, -0x1.ae600aca92c64p-26);
  s = kfma(s, z, 0x1.71de379654304p-19);
  s = kfma(s, z, -0x1.a01a019e83816p-13);
  s = kfma(s, z, 0x1.1111111110bb2p-7);
  s = kfma(s, z, -0x1.5555555555555p-3);
  s = fma(r * z, s, r);
  double c = -0x1.907d8f29fe831p-37;
  c = kfma(c, z, 0x1.1eeb68cd22f56p-29);
  c = kfma(c, z, -0x1.27e4fa17bf139p-22);
  c = kfma(c, z, 0x1.a01a019f4e9b4p-16);
  c = kfma(c, z, -0x1.6c16c16c16967p-10);
  c = kfma(c, z, 0x1.5555555555555p-5);
  const double h = fma(-0.5, z, 1.0);  // 1 - z/2 and its rounding error
  c = h + fma(z * z, c, fma(-0.5, z, 1.0 - h));
  const double a = (q & 1) ? c : s, b = (q & 1) ? s : c;
  *sp = (q & 2) ? -a : a;
  *cp = ((q + 1) & 2) ? -b : b;
}

// log(1 + f) + e ln 2 for 1 + f in [sqrt(1/2), sqrt(2)]: with s = f / (2 + f),
// log(1 + f) = 2 atanh(s) = f - s (f - R(s^2)), R = 2 s^2 (1/3 + s^2 / 5 + ...)
M64_FN double log_poly(double f, double e) {
  const double s = fdiv(f, 2.0 + f), z = s * s;
  double p = 0x1.2b5f6ba5f7c76p-3;
  p = kfma(p, z, 0x1.39fdccad06992p-3);
  p = kfma(p, z, 0x1.7462b91d6e050p-3);
  p = kfma(p, z, 0x1.c71c62d5dea59p-3);
  p = kfma(p, z, 0x1.2492492dfd8bfp-2);
  p = kfma(p, z, 0x1.9999999995273p-2);
  p = kfma(p, z, 0x1.5555555555558p-1);
  const double t = fma(-s, fma(-p, z, f), e * 0x1.abc9e3b39803fp-56);
  return fma(e, 0x1.62e42fefa39efp-1, f + t);
}

M64_FN double flog(double x) {
  double m = M64_MANT(x);
  int e = M64_EXPO(x);
  const bool lo = m < 0.70710678118654752;
  m = lo ? m + m : m;
  e -= lo ? 1 : 0;
  const double v = log_poly(m - 1.0, (double)e);
  return x > 0.0 ? (x < INFINITY ? v : x) : (x == 0.0 ? -INFINITY : NAN);  // x NaN: not > 0, not == 0
}

// log(1 + t), t >= -1: the rounding error of 1 + t is carried into the reduced argument
M64_FN double flog1p(double t) {
  const double u = 1.0 + t, bp = u - 1.0, c = (1.0 - (u - bp)) + (t - bp);  // 1 + t = u + c
  double m = M64_MANT(u);
  int e = M64_EXPO(u);
  const bool lo = m < 0.70710678118654752;
  m = lo ? m + m : m;
  e -= lo ? 1 : 0;
  const double v = log_poly((m - 1.0) + ldexp(c, -e), (double)e);
  return u > 0.0 ? (u < INFINITY ? v : u) : (u == 0.0 ? -INFINITY : NAN);
}

M64_FN double fatan2(double y, double x) {
  const double ax = fabs(x), ay = fabs(y), mx = fmax(ax, ay), mn = fmin(ax, ay);
  const bool hi = mn > 0.41421356237309503 * mx;  // beyond tan(pi/8): atan t = pi/4 + atan((t - 1) / (t + 1))
  const int sc = 1 - M64_EXPO(mx);                 // the quotient of operands scaled to mx in [1, 2)
  const double sm = ldexp(mx, sc), sn = ldexp(mn, sc);
  double t = fdiv(hi ? sn - sm : sn, hi ? sn + sm : sm);
  t = mx == 0.0 ? 0.0 : t;
  t = mn == INFINITY ? 0.0 : (mx == INFINITY ? 0.0 : t);  // both infinite: pi/4 exactly (hi is false, set below)
  const double z = t * t;
  double p = -0x1.3a2b6e74f00e0p-6;
  p = kfma(p, z, 0x1.4160318e023c6p-5);
  p = kfma(p, z, -0x1.a098b9c8d8226p-5);
  p = kfma(p, z, 0x1.dfe61e3086617p-5);
  p = kfma(p, z, -0x1.10fa753389c37p-4);
  p = kfma(p, z, 0x1.3b1262d901bc4p-4);
  p = kfma(p, z, -0x1.745d0b26b4a39p-4);
  p = kfma(p, z, 0x1.c71c718531360p-4);
  p = kfma(p, z, -0x1.24924924360c8p-3);
  p = kfma(p, z, 0x1.999999999934ap-3);
  p = kfma(p, z, -0x1.5555555555555p-2);
  double a = fma(t * z, p, t);
  const bool quarter = hi || (mn == INFINITY);
  a = quarter ? 0.78539816339744831 + (a + 3.0616169978683830e-17) : a;
  a = ay > ax ? 1.5707963267948966 - (a - 6.1232339957367660e-17) : a;
  a = std::signbit(x) ? 3.1415926535897931 - (a - 1.2246467991473532e-16) : a;
  a = copysign(a, y);
  return (x != x || y != y) ? x + y : a;
}

// remainder(y, 2 pi) with 2 pi rounded to float64: y - 2 pi rint(y / 2 pi), an exact difference
// for |y| < 2^50.  From 2^30 on, where the rounded quotient can be off by one near its halves,
// multiples 2^e n of 2 pi, n < 2^48, are taken off first, exactly as well.
M64_FN double wrap_2pi(double y) {
  while (fabs(y) >= 0x1p30 && fabs(y) < INFINITY) {
    const int x = M64_EXPO(y) - 50, e = x > 0 ? x : 0;
    y = fma(-rint(ldexp(y, -e) * 0.15915494309189535), ldexp(6.283185307179586477, e), y);
  }
  return fma(-rint(y * 0.15915494309189535), 6.283185307179586477, y);
}

}  // namespace m64
