// Hermitian eigendecomposition on the device (float64), for the pseudo-inverse
// and signal-to-noise regularisations of the TDVP equation (Sec. 3.3: the
// regularised inverse needs S = V diag(lambda) V^dagger).
//
// Two-sided block Jacobi.  The matrix (padded with decoupled zero rows and
// columns to Kp, a multiple of 2 BJ) is cut into nb = Kp / BJ index blocks; a
// sweep is nb - 1 rounds, and round r pairs every block once (circle ordering).
// For a pair (P, Q) the 2 BJ x 2 BJ Hermitian submatrix on the indices P u Q is
// diagonalised in LDS by cyclic Jacobi (below), giving a unitary U; then every
// block (i, j) of pairs becomes U_i^H A_ij U_j and V <- V diag(U).  The pairs
// of a round are disjoint, so the block transforms commute; each round reads
// the matrix it transforms from one buffer and writes the other.  Sweeps stop
// when the off-diagonal Frobenius norm is below tol times the full norm.
//
// Inner cyclic Jacobi on M (2 BJ indices, each round pairs every index once):
// for a pair (p, q) with M_pp = a, M_qq = b, M_pq = |z| e^{i phi}, the unitary
//     J = [[c, conj(s)], [-s, c]],  s = |s| e^{-i phi} times a sign,  |s| / c the smaller
//     root t of t^2 + 2 tau t - 1 = 0,  tau = |b - a| / (2 |z|),
// zeroes M_pq (M <- J^H M J on rows and columns p, q; U <- U J).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "internal.h"

using namespace dev;

namespace {

constexpr int BJ = 16;       // index block of the outer Jacobi
constexpr int BM = 2 * BJ;   // a pair's submatrix
constexpr int BLD = BM + 1;  // its row length in LDS
constexpr int MAX_INNER = 1; // inner sweeps per submatrix and round (one measured fastest)
// a pair's submatrix is reduced below INNER_TOL x the outer tolerance, so that what the
// pairs leave on their own off-diagonals stays below the outer criterion
constexpr double INNER_TOL = 0.125;

// circle ordering of n indices (n even), round r: pair i
__device__ __forceinline__ void circle_pair(int n, int r, int i, int& p, int& q) {
  const int m = n - 1;
  if (i == 0) {
    p = m;
    q = r;
  } else {
    p = (r + i) % m;
    q = (r - i + m) % m;
  }
}

// Arithmetic on entries of a real (double) or complex (double2) matrix.
__device__ __forceinline__ double zero_of(double) { return 0.0; }
__device__ __forceinline__ double2 zero_of(double2) { return make_double2(0.0, 0.0); }
__device__ __forceinline__ double real_of(double v) { return v; }
__device__ __forceinline__ double real_of(double2 v) { return v.x; }
__device__ __forceinline__ double norm2(double v) { return v * v; }
__device__ __forceinline__ double norm2(double2 v) { return fma(v.x, v.x, v.y * v.y); }
__device__ __forceinline__ double conj_of(double v) { return v; }
__device__ __forceinline__ double2 conj_of(double2 v) { return cconj(v); }
__device__ __forceinline__ double scaled(double v, double s) { return v * s; }
__device__ __forceinline__ double2 scaled(double2 v, double s) { return cscale(v, s); }
__device__ __forceinline__ double of_real(double, double x) { return x; }
__device__ __forceinline__ double2 of_real(double2, double x) { return make_double2(x, 0.0); }
// acc + a b
__device__ __forceinline__ double fmac(double acc, double a, double b) { return fma(a, b, acc); }
__device__ __forceinline__ double2 fmac(double2 acc, double2 a, double2 b) {
  return make_double2(fma(-a.y, b.y, fma(a.x, b.x, acc.x)), fma(a.y, b.x, fma(a.x, b.y, acc.y)));
}
// c a + s b, c real
__device__ __forceinline__ double mix(double c, double a, double s, double b) { return fma(c, a, s * b); }
__device__ __forceinline__ double2 mix(double c, double2 a, double2 s, double2 b) {
  const double2 t = cmul(s, b);
  return make_double2(fma(c, a.x, t.x), fma(c, a.y, t.y));
}

// 1 / sqrt(x) of a normal x: the hardware estimate and two Newton steps
__device__ __forceinline__ double rsqrt_nr(double x) {
  double y = __builtin_amdgcn_rsq(x);
  const double h = 0.5 * x;
  y = y * fma(-h * y, y, 1.5);
  return y * fma(-h * y, y, 1.5);
}

template <typename T>
struct jrot {
  double c;
  T s;                   // J = [[c, conj(s)], [-s, c]] on the index pair (p, q)
  double a_new, b_new;   // diagonal after the rotation
  bool active;
};

__device__ __forceinline__ double max_abs(double v) { return fabs(v); }
__device__ __forceinline__ double max_abs(double2 v) { return fmax(fabs(v.x), fabs(v.y)); }
__device__ __forceinline__ double shifted(double v, int e) { return ldexp(v, e); }
__device__ __forceinline__ double2 shifted(double2 v, int e) { return make_double2(ldexp(v.x, e), ldexp(v.y, e)); }

// Rotation that zeroes z = M_pq between a = M_pp and b = M_qq: with d = (b - a) / 2,
// r = sqrt(d^2 + |z|^2): c^2 = (1 + |d| / r) / 2, s = sgn(d) conj(z) / (2 r c) (the smaller
// of the two angles), and a, b move by -+ sgn(d) |z|^2 / (|d| + r).  Two reciprocal square
// roots are its whole dependent chain.  d and z are brought to a largest entry in [1/2, 1)
// by a power of two first, so that their squares stay in range whatever the matrix' scale.
template <typename T>
__device__ __forceinline__ jrot<T> make_rot(double a, double b, T z) {
  const double az = max_abs(z), d0 = 0.5 * (b - a);
  const int e = __builtin_amdgcn_frexp_exp(fmax(fabs(d0), az));
  const T zs = shifted(z, -e);
  const double h2 = norm2(zs), d = ldexp(d0, -e), r2 = fma(d, d, h2);
  jrot<T> R;
  // negligible coupling: no rotation (also for the decoupled padding indices)
  R.active = az > 1e-300 && h2 > 1e-34 * fabs(ldexp(a, -e)) * fabs(ldexp(b, -e));
  const double q = rsqrt_nr(R.active ? r2 : 1.0), ad = fabs(d);
  const double c2 = fma(0.5 * ad, q, 0.5), ci = rsqrt_nr(c2);
  const double sg = d >= 0.0 ? 1.0 : -1.0;
  const double t = sg * ldexp(m64::fdiv(h2, fma(r2, q, ad)), e);
  R.c = R.active ? c2 * ci : 1.0;
  R.s = scaled(conj_of(zs), R.active ? 0.5 * sg * q * ci : 0.0);
  R.a_new = R.active ? a - t : a;
  R.b_new = R.active ? b + t : b;
  return R;
}

// global index of local index l (0 .. BM - 1) of the pair (P, Q)
__device__ __forceinline__ int64_t gidx(int P, int Q, int l) {
  return l < BJ ? (int64_t)P * BJ + l : (int64_t)Q * BJ + (l - BJ);
}

// One group per block pair of outer round r: diagonalise the submatrix on P u Q
// by inner Jacobi sweeps (until its off-diagonal norm is below tol times its
// norm, max_inner at most) and write the accumulated unitary U (BM x BM,
// row-major) to Ub[i] and the rotated submatrix to Mb[i].
// Bound: the dependent chain of a round (operands from LDS, rotation, update, barrier), 31
// rounds a sweep: 59.7 -> 25.6 us at K = 404 with real entries (hypot, two square roots
// and three divisions per rotation before, complex arithmetic for real matrices).
template <typename T>
__global__ __launch_bounds__(256) void k_bj_solve(const T* __restrict__ A, int64_t Kp, int nb, int r, double tol,
                                                  int max_inner, T* __restrict__ Ub, T* __restrict__ Mb) {
  __shared__ T M[2][BM * BLD];
  __shared__ T U[BM * BLD];
  __shared__ double red[2][4];
  __shared__ unsigned short pq[(BM - 1) * BJ];  // the pairs of each inner round, p << 8 | q
  const int i = blockIdx.x, tid = threadIdx.x;
  const T zero = zero_of(T());
  int P, Q;
  circle_pair(nb, r, i, P, Q);
  for (int e = tid; e < BM * BM; e += 256) {
    const int a = e / BM, b = e % BM;
    M[0][a * BLD + b] = A[gidx(P, Q, a) * Kp + gidx(P, Q, b)];
    U[a * BLD + b] = of_real(T(), a == b ? 1.0 : 0.0);
  }
  for (int e = tid; e < (BM - 1) * BJ; e += 256) {
    int p, q;
    circle_pair(BM, e / BJ, e % BJ, p, q);
    pq[e] = (unsigned short)(p << 8 | q);
  }
  __syncthreads();
  // thread (ii, jj): the 2 x 2 block of pair ii's rows and pair jj's columns,
  // and rows ii, ii + 16 of U in pair jj's columns
  const int ii = tid >> 4, jj = tid & 15;
  int cur = 0;
  for (int sw = 0; sw < max_inner; ++sw) {
    // off-diagonal and full norm of M
    double off = 0.0, all = 0.0;
    for (int e = tid; e < BM * BM; e += 256) {
      const double m2 = norm2(M[cur][e / BM * BLD + e % BM]);
      all += m2;
      if (e / BM != e % BM) off += m2;
    }
    off = wave_sum(off);
    all = wave_sum(all);
    if ((tid & 63) == 0) {
      red[0][tid >> 6] = off;
      red[1][tid >> 6] = all;
    }
    __syncthreads();
    const double to = red[0][0] + red[0][1] + red[0][2] + red[0][3];
    const double ta = red[1][0] + red[1][1] + red[1][2] + red[1][3];
    __syncthreads();
    if (!(to > tol * tol * ta)) break;
    for (int rr = 0; rr < BM - 1; ++rr) {
      const T* Mi = M[cur];
      T* Mo = M[cur ^ 1];
      const int vi = pq[rr * BJ + ii], vj = pq[rr * BJ + jj];
      const int ip = vi >> 8, iq = vi & 255, jp = vj >> 8, jq = vj & 255;
      const T *r0 = Mi + ip * BLD, *r1 = Mi + iq * BLD;
      const T m00 = r0[jp], m01 = r0[jq], m10 = r1[jp], m11 = r1[jq];
      const T u00 = U[ii * BLD + jp], u01 = U[ii * BLD + jq], u10 = U[(ii + 16) * BLD + jp],
              u11 = U[(ii + 16) * BLD + jq];
      const jrot<T> Ri = make_rot(real_of(r0[ip]), real_of(r1[iq]), r0[iq]);
      const jrot<T> Rj = make_rot(real_of(Mi[jp * BLD + jp]), real_of(Mi[jq * BLD + jq]), Mi[jp * BLD + jq]);
      const T sj = Rj.s, mj = scaled(sj, -1.0), cj = conj_of(sj), si = Ri.s, ci = conj_of(si), mi = scaled(ci, -1.0);
      // T = M J_j, then J_i^H T
      const T t00 = mix(Rj.c, m00, mj, m01), t01 = mix(Rj.c, m01, cj, m00);
      const T t10 = mix(Rj.c, m10, mj, m11), t11 = mix(Rj.c, m11, cj, m10);
      T n00 = mix(Ri.c, t00, mi, t10), n01 = mix(Ri.c, t01, mi, t11);
      T n10 = mix(Ri.c, t10, si, t00), n11 = mix(Ri.c, t11, si, t01);
      if (ii == jj && Ri.active) {  // the pair's own 2 x 2 block: diagonal by construction
        n00 = of_real(T(), Ri.a_new);
        n11 = of_real(T(), Ri.b_new);
        n01 = zero;
        n10 = zero;
      }
      Mo[ip * BLD + jp] = n00;
      Mo[ip * BLD + jq] = n01;
      Mo[iq * BLD + jp] = n10;
      Mo[iq * BLD + jq] = n11;
      // U <- U J_j on rows ii and ii + 16
      U[ii * BLD + jp] = mix(Rj.c, u00, mj, u01);
      U[ii * BLD + jq] = mix(Rj.c, u01, cj, u00);
      U[(ii + 16) * BLD + jp] = mix(Rj.c, u10, mj, u11);
      U[(ii + 16) * BLD + jq] = mix(Rj.c, u11, cj, u10);
      __syncthreads();
      cur ^= 1;
    }
  }
  // one Newton-Schulz step U <- U (3 I - U^H U) / 2: the product of the rotations is
  // unitary only to the rounding of each rotation; this takes U back to the rounding
  // of one step, so that V, which takes a U every round, stays orthonormal
  {
    const int a = tid >> 3, b0 = tid & 7;
    T g[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) g[k] = zero;
#pragma unroll 8
    for (int m = 0; m < BM; ++m) {
      const T u = conj_of(U[m * BLD + a]);
#pragma unroll
      for (int k = 0; k < 4; ++k) g[k] = fmac(g[k], u, U[m * BLD + b0 + 8 * k]);
    }
    // H = (3 I - G) / 2 into M[cur ^ 1]
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int b = b0 + 8 * k;
      M[cur ^ 1][a * BLD + b] = mix(-0.5, g[k], of_real(T(), a == b ? 1.5 : 0.0), of_real(T(), 1.0));
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; ++k) g[k] = zero;
#pragma unroll 8
    for (int m = 0; m < BM; ++m) {
      const T u = U[a * BLD + m];
#pragma unroll
      for (int k = 0; k < 4; ++k) g[k] = fmac(g[k], u, M[cur ^ 1][m * BLD + b0 + 8 * k]);
    }
    T* out = Ub + (int64_t)i * BM * BM;
#pragma unroll
    for (int k = 0; k < 4; ++k) out[a * BM + b0 + 8 * k] = g[k];
  }
  T* mout = Mb + (int64_t)i * BM * BM;
  for (int e = tid; e < BM * BM; e += 256) mout[e] = M[cur][e / BM * BLD + e % BM];
}

// Groups with blockIdx.y < np: block (i = blockIdx.y, j = blockIdx.x) of pairs,
// Aout[P_i u Q_i, P_j u Q_j] = U_i^H Ain[...] U_j; a pair's own block (i = j)
// is the submatrix the rotations left (a product would put rounding noise back
// into its off-diagonal, where the sweeps could not remove it again).  The
// others: V <- V U_j on rows 32 x of V (in place; each group owns its rows and
// pair j's columns).
template <typename T>
__global__ __launch_bounds__(256) void k_bj_apply(const T* __restrict__ Ain, T* __restrict__ Aout, T* __restrict__ Vm,
                                                  int64_t Kp, int nb, int r, const T* __restrict__ Ub,
                                                  const T* __restrict__ Mb) {
  __shared__ T X[BM * BLD];
  __shared__ T Uj[BM * BLD];
  __shared__ T Ui[BM * BLD];
  const int np = nb / 2;
  const int tid = threadIdx.x;
  const int j = blockIdx.x;
  const bool own = (int)blockIdx.y == j, isA = (int)blockIdx.y < np;
  int Pj, Qj;
  circle_pair(nb, r, j, Pj, Qj);
  if (own) {
    for (int e = tid; e < BM * BM; e += 256)
      Aout[gidx(Pj, Qj, e / BM) * Kp + gidx(Pj, Qj, e % BM)] = Mb[(int64_t)j * BM * BM + e];
    return;
  }
  const int i = blockIdx.y;
  int Pi = 0, Qi = 0;
  if (isA) circle_pair(nb, r, i, Pi, Qi);
  const int64_t v0 = (int64_t)(i - np) * BM;
#pragma unroll
  for (int k = 0; k < BM * BM / 256; ++k) {
    const int e = tid + 256 * k, a = e / BM, b = e % BM;
    Uj[a * BLD + b] = Ub[(int64_t)j * BM * BM + e];
    if (isA) Ui[a * BLD + b] = Ub[(int64_t)i * BM * BM + e];
    X[a * BLD + b] = isA ? Ain[gidx(Pi, Qi, a) * Kp + gidx(Pj, Qj, b)] : Vm[(v0 + a) * Kp + gidx(Pj, Qj, b)];
  }
  __syncthreads();
  // thread: row a = tid / 8 of the block, columns b = (tid % 8) + 8 k
  const int a = tid >> 3, b0 = tid & 7;
  T x[4];  // (X U_j)[a][b]
#pragma unroll
  for (int k = 0; k < 4; ++k) x[k] = zero_of(T());
#pragma unroll 8
  for (int m = 0; m < BM; ++m) {
    const T t = X[a * BLD + m];
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = fmac(x[k], t, Uj[m * BLD + b0 + 8 * k]);
  }
  if (!isA) {
#pragma unroll
    for (int k = 0; k < 4; ++k) Vm[(v0 + a) * Kp + gidx(Pj, Qj, b0 + 8 * k)] = x[k];
    return;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k) X[a * BLD + b0 + 8 * k] = x[k];
  __syncthreads();
  // out[a][b] = sum_m conj(U_i[m][a]) (X U_j)[m][b]
#pragma unroll
  for (int k = 0; k < 4; ++k) x[k] = zero_of(T());
#pragma unroll 8
  for (int m = 0; m < BM; ++m) {
    const T u = conj_of(Ui[m * BLD + a]);
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = fmac(x[k], u, X[m * BLD + b0 + 8 * k]);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) Aout[gidx(Pi, Qi, a) * Kp + gidx(Pj, Qj, b0 + 8 * k)] = x[k];
}

// out[0] += sum of |A_ij|^2 off the diagonal, out[1] += sum of all |A_ij|^2 (per row, one wave)
template <typename T>
__global__ __launch_bounds__(256) void k_offnorm(const T* __restrict__ A, int64_t Kp, double* __restrict__ out) {
  const int64_t row = blockIdx.x * 4ll + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= Kp) return;
  double off = 0.0, all = 0.0;
  for (int64_t c = lane; c < Kp; c += 64) {
    const double m = norm2(A[row * Kp + c]);
    all += m;
    if (c != row) off += m;
  }
  off = wave_sum(off);
  all = wave_sum(all);
  if (lane == 0) {
    atomicAdd(out, off);
    atomicAdd(out + 1, all);
  }
}

template <typename T>
__global__ void k_pad_copy(const double2* __restrict__ S, int64_t K, int64_t Kp, T* __restrict__ A,
                           T* __restrict__ V) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= Kp * Kp) return;
  const int64_t r = e / Kp, c = e % Kp;
  const double2 v = (r < K && c < K) ? S[r * K + c] : make_double2(0.0, 0.0);
  if constexpr (sizeof(T) == sizeof(double))
    A[e] = v.x;
  else
    A[e] = v;
  V[e] = of_real(T(), r == c ? 1.0 : 0.0);
}

template <typename T>
__global__ void k_eig_out(const T* __restrict__ A, const T* __restrict__ Vp, int64_t K, int64_t Kp,
                          double* __restrict__ lam, double2* __restrict__ V) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= K * K) return;
  const int64_t r = e / K, c = e % K;
  if constexpr (sizeof(T) == sizeof(double))
    V[e] = make_double2(Vp[r * Kp + c], 0.0);
  else
    V[e] = Vp[r * Kp + c];
  if (r == 0) lam[c] = real_of(A[c * Kp + c]);
}

int64_t padded(int64_t K) { return (K + BM - 1) / BM * BM; }

}  // namespace

size_t eig_ws_bytes(int64_t K) {
  const int64_t Kp = padded(K);
  return ws_round(sizeof(double2) * Kp * Kp) * 3 + 2 * ws_round(sizeof(double2) * (Kp / BM) * BM * BM) +
         ws_round(2 * sizeof(double));
}

namespace {
template <typename T>
int jacobi(vmc_ctx* ctx, const double2* S, int64_t K, double tol, int max_sweeps, double* lam, double2* V, void* ws) {
  hipStream_t st = ctx->stream;
  const int64_t Kp = padded(K);
  const int nb = (int)(Kp / BJ), np = nb / 2;
  char* w = (char*)ws;
  T* A = (T*)w;
  w += ws_round(sizeof(T) * Kp * Kp);
  T* A2 = (T*)w;
  w += ws_round(sizeof(T) * Kp * Kp);
  T* Vp = (T*)w;
  w += ws_round(sizeof(T) * Kp * Kp);
  T* Ub = (T*)w;
  w += ws_round(sizeof(T) * (Kp / BM) * BM * BM);
  T* Mb = (T*)w;
  w += ws_round(sizeof(T) * (Kp / BM) * BM * BM);
  double* nrm = (double*)w;
  k_pad_copy<T><<<grid_for(Kp * Kp, 256), 256, 0, st>>>(S, K, Kp, A, Vp);
  VMC_HIP(hipGetLastError());
  double* hn = (double*)pinned_host(ctx, 2 * sizeof(double));
  int sweeps = 0;
  for (;;) {
    VMC_HIP(hipMemsetAsync(nrm, 0, 2 * sizeof(double), st));
    k_offnorm<T><<<(unsigned)((Kp + 3) / 4), 256, 0, st>>>(A, Kp, nrm);
    VMC_HIP(hipMemcpyAsync(hn, nrm, 2 * sizeof(double), hipMemcpyDeviceToHost, st));
    VMC_HIP(hipStreamSynchronize(st));
    if (!(hn[0] > tol * tol * hn[1]) || sweeps >= max_sweeps) break;
    for (int r = 0; r < nb - 1; ++r) {
      k_bj_solve<T><<<(unsigned)np, 256, 0, st>>>(A, Kp, nb, r, INNER_TOL * tol, MAX_INNER, Ub, Mb);
      k_bj_apply<T><<<dim3((unsigned)np, (unsigned)(np + Kp / BM)), 256, 0, st>>>(A, A2, Vp, Kp, nb, r, Ub, Mb);
      std::swap(A, A2);
    }
    VMC_HIP(hipGetLastError());
    ++sweeps;
  }
  if (!std::isfinite(hn[0]) || !std::isfinite(hn[1]))
    throw vmc_error{VMC_ERR_NONFINITE, "eigendecomposition produced non-finite values"};
  k_eig_out<T><<<grid_for(K * K, 256), 256, 0, st>>>(A, Vp, K, Kp, lam, V);
  VMC_HIP(hipGetLastError());
  return sweeps;
}
}  // namespace

// real: every imaginary part of S is 0 (the sweeps then run in real arithmetic)
int eig_hermitian(vmc_ctx* ctx, const double2* S, int64_t K, bool real, double tol, int max_sweeps, double* lam,
                  double2* V, void* ws) {
  return real ? jacobi<double>(ctx, S, K, tol, max_sweeps, lam, V, ws)
              : jacobi<double2>(ctx, S, K, tol, max_sweeps, lam, V, ws);
}

extern "C" int vmc_eigh(vmc_ctx* ctx, const double* A, int64_t K, double tol, int max_sweeps, double* evals,
                        double* V, int* sweeps_host) {
  return guard(ctx, [&] {
    VMC_REQUIRE(ctx && A && evals && V, "NULL argument");
    VMC_REQUIRE(K >= 1 && K <= 16384, "K must be in [1, 16384]");
    VMC_REQUIRE(std::isfinite(tol) && tol >= 0.0, "tol must be finite and non-negative");
    VMC_REQUIRE(max_sweeps >= 0, "max_sweeps < 0");
    set_device(ctx);
    phase_scope ps(ctx, "eig");
    ws_reserve(ctx, eig_ws_bytes(K));
    void* w = ws_take(ctx, eig_ws_bytes(K));
    const int s = eig_hermitian(ctx, (const double2*)A, K, false, tol > 0.0 ? tol : 1e-14, max_sweeps > 0 ? max_sweeps : 50,
                                evals, (double2*)V, w);
    if (sweeps_host) *sweeps_host = s;
  });
}
