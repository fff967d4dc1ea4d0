// Blocked right-looking Cholesky S~ = L L^H in float64 (lower triangle, row-major,
// in place) and the two triangular solves, block size 64.
//
// Two levels: 256-column panels, each factored as four 64-column blocks.
// Per 64-column block b:
//   k_chol_diag   one work-group factors the diagonal block in registers,
//                 writes L_bb, inverts it and writes L_bb^{-1} (dense
//                 64 x 64) to the Linv buffer;
//   k_zprod SOLVE rows below: L_rb = A_rb L_bb^{-H}, a complex GEMM on the
//                 float64 matrix cores (in place, one 64-row block per group);
//   k_zprod RECT  the rest of the panel's columns: A_rc -= L_rb L_cb^H.
// Per panel p, once its four blocks are done:
//   k_zprod RECT  lookahead: the next panel's columns -= L_rp L_cp^H;
//   k_zprod TRI   trailing update A_rc -= L_rp L_cp^H (reduction depth 256) on
//                 the lower 64 x 64 tiles of the rest of the trailing matrix,
//                 on a second stream, overlapping the next panel's
//                 factorisation; the trailing matrix is read and written once
//                 per 256 columns.
// The complex products P conj(Q) take three real products per term (Gauss's
// identity, as in the 3M complex GEMM): with A = sum Pr Qr, B = sum Pi Qi and
// C = sum (Pr + Pi)(Qr - Qi), held in three accumulators at the same lanes,
//   Re = A + B,   Im = C - A + B,
// so a 16x16 complex block costs three float64 MFMAs per 4 reduction columns
// instead of four; the error bound of Im grows by at most a factor of about 2.
// A non-positive pivot sets the fail index; every later kernel then exits at
// once.  The upper triangle of S~ is never written.
//
// Triangular solves: one launch per direction, one group per 64-row block,
// blocks handed over through ready flags in the order of the solve.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "internal.h"

using namespace dev;

namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));

constexpr int CB = 64;  // block size

// Factor and invert the diagonal block at kb0 (nb <= 64 valid rows/cols; the
// rest is padded with the identity).
// Right-looking elimination on the unscaled Schur complement and the inverse
// of the unit-lower factor together, one barrier per column j.  With
// f_r = A_rj / A_jj (the multiplier of row r, which equals L_rj / L_jj):
//   A_rc -= f_r conj(A_cj)   for j < c <= r   (elimination),
//   B_rc -= f_r B_jc         for c <= j < r   (B = I at the start; row j of B
//                                              is final after step j - 1).
// An entry (r, c) is A's up to step c, which reads it last, and B's from then
// on, so one register holds both and a second keeps A_rc for the factor:
// L_rc = A_rc / sqrt(d_c), L_cc = sqrt(d_c) and L^{-1}_rc = B_rc / sqrt(d_r),
// with the pivots d_j = A_jj.  Thread (ty, tx) of 16 x 16 holds rows ty + 16 a,
// columns tx + 16 b <= row; the owners of column j and row j publish the vectors
// F_r = A_rj and W_c = conj(A_cj) (c > j), 1 (c = j), B_jc (c < j), and every
// step is v_rc -= (F_r / d) W_c.
// Bound: 64 times the path from the update of column j + 1 over LDS and the
// barrier to the reciprocal and the next update (entries in LDS before, read and
// written each step by 512 threads): 37 us a block instead of 59 (K = 1 529:
// the factorisation 2.43 -> 1.91 ms).
__device__ __forceinline__ double recip(double d) {
  double x = __builtin_amdgcn_rcp(d);
  x = fma(x, fma(-d, x, 1.0), x);
  return fma(x, fma(-d, x, 1.0), x);
}

__global__ __launch_bounds__(256) void k_chol_diag(double2* __restrict__ A, int64_t K, int64_t kb0, int nb,
                                                   double2* __restrict__ Linv, long long* __restrict__ fail,
                                                   double* __restrict__ pivmin) {
  __shared__ double2 F[2][CB], W[2][CB];
  __shared__ double dp[CB], sq[CB], isq[CB];
  if (*fail >= 0) return;
  const int tid = threadIdx.x, ty = tid >> 4, tx = tid & 15;
  double2 v[4][4], lr[4][4];  // entries (a, b), b <= a
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b <= a; ++b) {
      const int r = ty + 16 * a, c = tx + 16 * b;
      v[a][b] = make_double2(r == c ? 1.0 : 0.0, 0.0);
      if (c <= r && r < nb) v[a][b] = A[(kb0 + r) * K + kb0 + c];
      lr[a][b] = v[a][b];
    }
  // column and row j = 16 jb + jj of the entries updated through step j - 1
  auto publish = [&](auto jbc, int jj) {
    constexpr int jb = decltype(jbc)::value;
    const int buf = jj & 1;
    if (tx == jj) {
#pragma unroll
      for (int a = jb; a < 4; ++a) {
        const int r = ty + 16 * a;
        if (a > jb || ty > jj) {
          F[buf][r] = v[a][jb];
          W[buf][r] = cconj(v[a][jb]);
        } else if (ty == jj) {
          dp[r] = v[a][jb].x;
          W[buf][r] = make_double2(1.0, 0.0);
        }
      }
    }
    if (ty == jj) {
#pragma unroll
      for (int b = 0; b <= jb; ++b)
        if (b < jb || tx < jj) W[buf][tx + 16 * b] = v[jb][b];
    }
  };
  int bad = -1;
  double pmin = INFINITY;
  auto block = [&](auto jbc) {
    constexpr int jb = decltype(jbc)::value;
#pragma unroll 2
    for (int jj = 0; jj < 16; ++jj) {
      const int j = 16 * jb + jj, buf = jj & 1;
      __syncthreads();
      const double d = dp[j];  // the same value in every thread
      if (j < nb) {
        pmin = fmin(pmin, d);
        if (!(d > 0.0)) {
          bad = j;
          return;
        }
      }
      const double id = recip(d);
      double2 w[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) w[b] = W[buf][tx + 16 * b];
#pragma unroll
      for (int a = jb; a < 4; ++a) {
        if (a == jb && ty <= jj) continue;  // rows up to j are final
        const double2 f = cscale(F[buf][ty + 16 * a], id);
        if (tx == jj) {
          lr[a][jb] = v[a][jb];
          v[a][jb] = make_double2(0.0, 0.0);
        }
#pragma unroll
        for (int b = 0; b <= a; ++b) v[a][b] = csub(v[a][b], cmul(f, w[b]));
      }
      if (jj < 15) {
        publish(jbc, jj + 1);
      } else if constexpr (jb < 3) {
        publish(std::integral_constant<int, jb + 1>{}, 0);
      }
    }
  };
  publish(std::integral_constant<int, 0>{}, 0);
  block(std::integral_constant<int, 0>{});
  if (bad < 0) block(std::integral_constant<int, 1>{});
  if (bad < 0) block(std::integral_constant<int, 2>{});
  if (bad < 0) block(std::integral_constant<int, 3>{});
  if (tid == 0) {
    pivmin[kb0 / CB] = pmin;
    if (bad >= 0) *fail = kb0 + bad;
  }
  if (bad >= 0) return;  // uniform: every thread saw the same pivot
  if (tid < CB) {
    const double t = sqrt(dp[tid]);
    sq[tid] = t;
    isq[tid] = 1.0 / t;
  }
  __syncthreads();
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int r = ty + 16 * a, c = tx + 16 * b;
      double2 xv = make_double2(0.0, 0.0);
      if (c < r) xv = cscale(v[a][b <= a ? b : a], isq[r]);
      if (c == r) xv = make_double2(isq[r], 0.0);
      if (c <= r && r < nb)
        A[(kb0 + r) * K + kb0 + c] = r == c ? make_double2(sq[c], 0.0) : cscale(lr[a][b <= a ? b : a], isq[c]);
      Linv[r * CB + c] = xv;
    }
}

struct zargs {
  double2* S;
  int64_t K;
  int64_t kb0;   // first panel column of the reduction
  int depth;     // valid panel columns (reduction length)
  int64_t rbase; // first output row
  int64_t cbase; // first output column
  int64_t cend;  // one past the last output column (RECT)
  int nct;       // column tiles (RECT); tile rows of the triangle (TRI)
  int sd;        // side of the squares of tiles (TRI)
  const double2* Linv;
  const long long* fail;
};

// The panel's and the trailing matrix' products on 64 x 64 tiles:
//   SOLVE  S[R][kb0 + c] = sum_m S[R][kb0 + m] conj(Linv[c][m]), R >= rbase (in place; depth 64)
//   RECT   S[R][C] -= sum_m S[R][kb0 + m] conj(S[C][kb0 + m]), R >= rbase, cbase <= C < cend, C <= R
//   TRI    the same for the lower triangle from (rbase, rbase) on
// The operands go straight from memory to LDS, eight columns a stage, two stages: row r of a
// tile is 128 bytes, its 16-byte entry of column m at place m ^ ((r / 2) % 8), so that the 16
// rows a fragment reads at one column fall on 16 different groups of banks.  A stage's
// fragments are read before the next stage's loads are issued: the compiler makes an LDS read
// wait for every load into LDS before it.  TRI tiles go out in squares of sd x sd per XCD,
// whose 2 sd operand rows meet in its L2.
// Bound: the matrix cores (62 ms of products at K = 16 704), and towards the end the panel's
// chain, whose kernels wait for a place beside the TRI launch.  Without staging registers
// three groups fit a compute unit, in any mix of the modes.  K = 16 704: all TRI launches 88
// -> 74 ms, the whole factorisation 95.1 -> 81.7 ms; K = 1 529 1.89 -> 1.68 ms (operands
// through registers, two groups per compute unit, one row of tiles after the other per XCD
// before).  TRI held to two groups per compute unit, to leave a place for the panel: 84.4 ms.
constexpr int ZS = 8;  // columns per stage

typedef __attribute__((address_space(3))) void* lptr_t;

enum { SOLVE, RECT, TRI };

template <int MODE>
__global__ __launch_bounds__(256, 3) void k_zprod(zargs a) {
  __shared__ double2 Ps[2][CB * ZS];
  __shared__ double2 Qs[2][CB * ZS];
  if (*a.fail >= 0) return;
  const int64_t K = a.K;
  int64_t r0, c0;
  if (MODE == SOLVE) {
    r0 = a.rbase + (int64_t)blockIdx.x * CB;
    c0 = 0;
  } else if (MODE == RECT) {
    r0 = a.rbase + (int64_t)(blockIdx.x / a.nct) * CB;
    c0 = a.cbase + (int64_t)(blockIdx.x % a.nct) * CB;
  } else {
    const int sd = a.sd, j = blockIdx.x / 8;
    const int64_t sq = (int64_t)(j / (sd * sd)) * 8 + blockIdx.x % 8;
    int sr = (int)((sqrt(8.0 * (double)sq + 1.0) - 1.0) * 0.5);
    while ((int64_t)(sr + 1) * (sr + 2) / 2 <= sq) ++sr;
    while ((int64_t)sr * (sr + 1) / 2 > sq) --sr;
    const int sc = (int)(sq - (int64_t)sr * (sr + 1) / 2), in = j % (sd * sd);
    const int tr = sr * sd + in / sd, tc = sc * sd + in % sd;
    if (tr >= a.nct || tc > tr) return;
    r0 = a.rbase + (int64_t)tr * CB;
    c0 = a.rbase + (int64_t)tc * CB;
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave >> 1, wc = wave & 1;
  const int li = lane & 15, lk = lane >> 4;
  doublex4 acc[2][2][3];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 3; ++q) acc[i][j][q] = doublex4{0.0, 0.0, 0.0, 0.0};

  // wave w loads rows 16 w .. 16 w + 15 of both tiles, eight rows per instruction; rows past
  // the matrix repeat its last one (their products are not written)
  const auto sp = __builtin_amdgcn_make_buffer_rsrc((void*)(a.S + r0 * K + a.kb0), 0, -1, 0x00027000);
  const auto sq = __builtin_amdgcn_make_buffer_rsrc(MODE == SOLVE ? (void*)a.Linv : (void*)(a.S + c0 * K + a.kb0), 0,
                                                    -1, 0x00027000);
  int vp[2], vq[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int r = 16 * wave + 8 * t + (lane >> 3), m = (lane & 7) ^ ((r >> 1) & 7);
    vp[t] = ((int)min((int64_t)r, K - 1 - r0) * (int)K + m) * 16;
    vq[t] = MODE == SOLVE ? (r * CB + m) * 16 : ((int)min((int64_t)r, K - 1 - c0) * (int)K + m) * 16;
  }
  auto load = [&](int st, int buf) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(sp, (lptr_t)(Ps[buf] + (16 * wave + 8 * t) * ZS), 16, vp[t],
                                               st * ZS * 16, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(sq, (lptr_t)(Qs[buf] + (16 * wave + 8 * t) * ZS), 16, vq[t],
                                               st * ZS * 16, 0, 0);
    }
  };
  const int nst = a.depth / ZS;
  load(0, 0);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  auto stage = [&](int st, auto bufc) {
    constexpr int buf = decltype(bufc)::value;
    double2 fa[2][2], fb[2][2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int at = (4 * ks + lk) ^ ((li >> 1) & 7);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        fa[ks][i] = Ps[buf][(wr * 32 + i * 16 + li) * ZS + at];
        fb[ks][i] = Qs[buf][(wc * 32 + i * 16 + li) * ZS + at];
      }
    }
    if (st + 1 < nst) load(st + 1, buf ^ 1);  // released by every wave at the last barrier
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      double sa[2], db[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        sa[i] = fa[ks][i].x + fa[ks][i].y;
        db[i] = fb[ks][i].x - fb[ks][i].y;
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          acc[i][j][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[ks][i].x, fb[ks][j].x, acc[i][j][0], 0, 0, 0);
          acc[i][j][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[ks][i].y, fb[ks][j].y, acc[i][j][1], 0, 0, 0);
          acc[i][j][2] = __builtin_amdgcn_mfma_f64_16x16x4f64(sa[i], db[j], acc[i][j][2], 0, 0, 0);
        }
    }
    __builtin_amdgcn_sched_barrier(0);  // the wait stays after the products
    __builtin_amdgcn_s_waitcnt(0);      // this wave's rows of the next stage have landed
    __syncthreads();                    // and every wave is done with this one
  };
  for (int st = 0; st < nst; st += 2) {
    stage(st, std::integral_constant<int, 0>{});
    if (st + 1 < nst) stage(st + 1, std::integral_constant<int, 1>{});
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t R = r0 + wr * 32 + i * 16 + lk + 4 * r, C = c0 + wc * 32 + j * 16 + li;
        const double re = acc[i][j][0][r] + acc[i][j][1][r];
        const double im = (acc[i][j][2][r] - acc[i][j][0][r]) + acc[i][j][1][r];
        if (MODE == SOLVE) {
          if (R < K) a.S[R * K + a.kb0 + C] = make_double2(re, im);
        } else if (R < K && C <= R && (MODE == TRI || C < a.cend)) {
          const double2 v = a.S[R * K + C];
          a.S[R * K + C] = make_double2(v.x - re, v.y - im);
        }
      }
}

__device__ __forceinline__ double2 shfl_xor2(double2 v, int o) {
  return make_double2(__shfl_xor(v.x, o, 64), __shfl_xor(v.y, o, 64));
}

// sum over the four lanes q = lane % 4 of a quad
__device__ __forceinline__ double2 quad_sum(double2 v) {
  v = cadd(v, shfl_xor2(v, 1));
  return cadd(v, shfl_xor2(v, 2));
}

// ---------------------------------------------------------------- solves --
// Each triangular solve is one launch with one group per 64-row block.  A group
// takes a ticket (an atomic counter) when it starts and solves the block with
// that rank in the order of the solve, so every block it waits for belongs to a
// group that started earlier: the waits end whatever the number of groups the
// device holds at once.  A block's solution is published by its group with a
// release store of a per-block ready flag; wave 0 of a consumer polls the flags
// (64 at a time, relaxed), then takes an acquire fence before it reads the
// solutions.  Off-diagonal products are accumulated in registers over all
// earlier blocks and reduced once, so the critical path per block is one flag
// hand-over, one 64-term update and the 64 x 64 product with L_bb^{-1}.
//
// sync layout (ints, zeroed before the forward solve): [0] forward ticket,
// [1, nblk] forward flags, [nblk + 1] backward ticket, [nblk + 2, 2 nblk + 1]
// backward flags, [2 nblk + 2] set when a wait exceeded its poll limit.
constexpr int kPollLimit = 1 << 22;  // polls (a global load and a short sleep each) before a wait gives up

__global__ void k_zero_ints(int* __restrict__ p, int n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0;
}

// Wave 0 of a group: wait until the flags of blocks j, j + d, j + 2d, ... up to
// (not including) `end` are set, at least block j; returns the first block
// past the leading run of set flags (d = +1 forward, -1 backward).
__device__ __forceinline__ int wait_ready(const int* __restrict__ flag, int j, int end, int d, int* __restrict__ err) {
  const int lane = threadIdx.x & 63;
  const int jl = j + d * lane;
  for (int polls = 0;; ++polls) {
    const bool in = d > 0 ? jl < end : jl > end;
    const int f = in ? __hip_atomic_load(flag + jl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    const unsigned long long m = __ballot(f != 0);
    const int n = ~m == 0ull ? 64 : __builtin_ctzll(~m);
    if (n > 0) {
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      return j + d * n;
    }
    if (polls >= kPollLimit) {  // never reached when every group runs to its end
      if (lane == 0) __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return j + d;
    }
    __builtin_amdgcn_s_sleep(2);
  }
}

// L y = rhs.  Group rank b: thread (r, q) = (tid / 4, tid % 4) accumulates
// sum_j L[R][64 j + m] y_j[m] over m = q, q + 4, ... for row R = 64 b + r
// (each quad reads 64 contiguous bytes of its row per load), then
// y_b = L_bb^{-1} (rhs_b - sum).  The row entries of the next two blocks are in
// flight while a block is applied (three register buffers in turn); L_bb^{-1}
// waits in LDS, so that two groups fit on a compute unit and every group of the
// launch is resident at once.
__global__ __launch_bounds__(256, 2) void k_fwd_chain(const double2* __restrict__ A, int64_t K, int nblk,
                                                      const double2* __restrict__ Linv, const double2* __restrict__ rhs,
                                                      double2* __restrict__ y, int* __restrict__ sync) {
  __shared__ int tk;
  __shared__ double2 li[CB * (CB + 1)];  // L_bb^{-1}, row stride 65
  __shared__ double2 yb[2][CB];
  __shared__ double2 rs[CB];
  __shared__ double2 ys[CB];
  const int tid = threadIdx.x;
  const int r = tid >> 2, q = tid & 3;
  if (tid == 0) tk = atomicAdd(sync, 1);
  __syncthreads();
  const int b = tk;
  int* flag = sync + 1;
  const int64_t R = (int64_t)b * CB + r;
  const bool row_ok = R < K;
  const int nb = (int)std::min<int64_t>(CB, K - (int64_t)b * CB);
  const double2 zero = make_double2(0.0, 0.0);
  const double2* Ar = A + (row_ok ? R : 0) * K + q;
  auto load_blk = [&](int j, double2(&v)[CB / 4]) {
#pragma unroll
    for (int t = 0; t < CB / 4; ++t) v[t] = row_ok ? Ar[(int64_t)j * CB + 4 * t] : zero;
  };
  double2 A0[CB / 4], A1[CB / 4], A2[CB / 4];
  if (b > 0) load_blk(0, A0);
  if (b > 1) load_blk(1, A1);
  const double2 rv = (row_ok && q == 0) ? rhs[R] : zero;
  for (int i = tid; i < CB * CB; i += 256) li[(i >> 6) * (CB + 1) + (i & 63)] = Linv[(size_t)b * CB * CB + i];
  double2 acc = zero;
  int ready = 0;  // wave 0: blocks [0, ready) are published
  // apply block j (entries in cur); the entries of block j + 2 go to pre
  auto step = [&](int j, double2(&cur)[CB / 4], double2(&pre)[CB / 4]) {
    if (tid < 64) {
      if (j >= ready) ready = wait_ready(flag, j, b, 1, sync + 2 * nblk + 2);
      yb[j & 1][tid] = y[(int64_t)j * CB + tid];  // block j < b is a full block
    }
    __syncthreads();
    if (j + 2 < b) load_blk(j + 2, pre);
#pragma unroll
    for (int t = 0; t < CB / 4; ++t) acc = cadd(acc, cmul(cur[t], yb[j & 1][4 * t + q]));
  };
  for (int j = 0; j < b; j += 3) {
    step(j, A0, A2);
    if (j + 1 < b) step(j + 1, A1, A0);
    if (j + 2 < b) step(j + 2, A2, A1);
  }
  acc = quad_sum(acc);
  if (q == 0) rs[r] = row_ok ? csub(rv, acc) : zero;
  __syncthreads();  // also orders the LDS copy of L_bb^{-1} before its reads
  double2 s = zero;
#pragma unroll
  for (int t = 0; t < CB / 4; ++t) {
    const int m = q + 4 * t;
    if (m <= r && m < nb) s = cadd(s, cmul(li[r * (CB + 1) + m], rs[m]));
  }
  s = quad_sum(s);
  if (q == 0) ys[r] = s;
  __syncthreads();
  if (tid < 64) {
    if (tid < nb) y[(int64_t)b * CB + tid] = ys[tid];
    __hip_atomic_store(flag + b, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// L^H x = y.  Group rank t solves block b = nblk - 1 - t: thread (w, c) =
// (tid / 64, tid % 64) accumulates sum_j sum_m conj(L[64 j + m][64 b + c]) x_j[m]
// over m = 16 w .. 16 w + 15 for j > b (each load reads 64 consecutive columns
// of one row), then x_b = L_bb^{-H} (y_b - sum).  Buffers as in the forward
// solve; here every step reads 64 rows not read before, so the two-block
// prefetch also covers their address-translation misses.
__global__ __launch_bounds__(256, 2) void k_bwd_chain(const double2* __restrict__ A, int64_t K, int nblk,
                                                      const double2* __restrict__ Linv, const double2* __restrict__ y,
                                                      double2* __restrict__ x, int* __restrict__ sync) {
  __shared__ int tk;
  __shared__ double2 li[CB * (CB + 1)];  // L_bb^{-1}, row stride 65
  __shared__ double2 xb[2][CB];
  __shared__ double2 part[4][CB];
  __shared__ double2 vs[CB];
  const int tid = threadIdx.x;
  const int w = tid >> 6, c = tid & 63;
  if (tid == 0) tk = atomicAdd(sync + nblk + 1, 1);
  __syncthreads();
  const int b = nblk - 1 - tk;
  int* flag = sync + nblk + 2;
  const int nb = (int)std::min<int64_t>(CB, K - (int64_t)b * CB);
  const double2 zero = make_double2(0.0, 0.0);
  auto nb_of = [&](int j) { return (int)std::min<int64_t>(CB, K - (int64_t)j * CB); };
  // column 64 b + c exists for every block b < nblk - 1, the only ones that load
  // (row addresses are wave-uniform: scalar bases plus the lane's column offset)
  const int wu = __builtin_amdgcn_readfirstlane(w);
  auto load_blk = [&](int j, double2(&v)[CB / 4]) {
    const int nbj = nb_of(j);
#pragma unroll
    for (int i = 0; i < CB / 4; ++i) {
      const int m = wu * (CB / 4) + i;
      const double2* row = A + ((int64_t)j * CB + m) * K + (int64_t)b * CB;
      v[i] = m < nbj ? cconj(row[c]) : zero;
    }
  };
  double2 A0[CB / 4], A1[CB / 4], A2[CB / 4];
  if (b < nblk - 1) load_blk(nblk - 1, A0);
  if (b < nblk - 2) load_blk(nblk - 2, A1);
  const double2 yv = tid < nb ? y[(int64_t)b * CB + tid] : zero;
  for (int i = tid; i < CB * CB; i += 256) li[(i >> 6) * (CB + 1) + (i & 63)] = Linv[(size_t)b * CB * CB + i];
  double2 acc = zero;
  int ready = nblk - 1;  // wave 0: blocks (ready, nblk) are published
  // apply block j (entries in cur); the entries of block j - 2 go to pre
  auto step = [&](int j, double2(&cur)[CB / 4], double2(&pre)[CB / 4]) {
    if (tid < 64) {
      if (j <= ready) ready = wait_ready(flag, j, b, -1, sync + 2 * nblk + 2);
      xb[j & 1][tid] = tid < nb_of(j) ? x[(int64_t)j * CB + tid] : zero;
    }
    __syncthreads();
    if (j - 2 > b) load_blk(j - 2, pre);
#pragma unroll
    for (int i = 0; i < CB / 4; ++i) acc = cadd(acc, cmul(cur[i], xb[j & 1][w * (CB / 4) + i]));
  };
  for (int j = nblk - 1; j > b; j -= 3) {
    step(j, A0, A2);
    if (j - 1 > b) step(j - 1, A1, A0);
    if (j - 2 > b) step(j - 2, A2, A1);
  }
  part[w][c] = acc;
  __syncthreads();  // also orders the LDS copy of L_bb^{-1} before its reads
  if (tid < 64)
    vs[tid] = tid < nb ? csub(yv, cadd(cadd(part[0][tid], part[1][tid]), cadd(part[2][tid], part[3][tid]))) : zero;
  __syncthreads();
  // x_b[c] = sum_{m >= c} conj(L_bb^{-1}[m][c]) v_b[m], wave w over m = w + 4 t
  double2 s = zero;
#pragma unroll
  for (int t = 0; t < CB / 4; ++t) {
    const int m = w + 4 * t;
    if (m >= c && m < nb) s = cadd(s, cmul(cconj(li[m * (CB + 1) + c]), vs[m]));
  }
  part[w][c] = s;  // every read of part above finished before the last barrier
  __syncthreads();
  if (tid < 64) {
    if (tid < nb) x[(int64_t)b * CB + tid] = cadd(cadd(part[0][tid], part[1][tid]), cadd(part[2][tid], part[3][tid]));
    __hip_atomic_store(flag + b, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
  }
}

}  // namespace

size_t chol_linv_bytes(int64_t K) { return sizeof(double2) * (size_t)((K + CB - 1) / CB) * CB * CB; }
int chol_block() { return CB; }

void chol_factor(vmc_ctx* ctx, double2* S, int64_t K, double2* Linv, long long* fail, double* pivmin) {
  hipStream_t st = ctx->stream;
  constexpr int PW = 256;  // panel width of the trailing update
  // Lookahead: after panel P_p is factored, the next panel's columns are
  // updated by P_p on the main stream, while the rest of the trailing matrix
  // (columns from the panel after next on) is updated on the auxiliary stream,
  // overlapping the factorisation of the next panel.  The only conflict is
  // the next lookahead (it writes columns the previous auxiliary update also
  // writes), so it waits for that update.
  hipStream_t aux = aux_stream(ctx);
  bool aux_busy = false;
  for (int64_t p0 = 0; p0 < K; p0 += PW) {
    const int64_t pend = std::min<int64_t>(K, p0 + PW);
    for (int64_t c0 = p0; c0 < pend; c0 += CB) {
      const int nb = (int)std::min<int64_t>(CB, K - c0);
      double2* Lb = Linv + (size_t)(c0 / CB) * CB * CB;
      k_chol_diag<<<1, 256, 0, st>>>(S, K, c0, nb, Lb, fail, pivmin);
      const int64_t rest = K - c0 - nb;
      if (rest <= 0) continue;
      zargs a{};
      a.S = S;
      a.K = K;
      a.kb0 = c0;
      a.depth = nb;
      a.rbase = c0 + nb;
      a.Linv = Lb;
      a.fail = fail;
      k_zprod<SOLVE><<<(unsigned)((rest + CB - 1) / CB), 256, 0, st>>>(a);
      if (c0 + nb < pend) {  // remaining columns of this panel
        a.cbase = c0 + nb;
        a.cend = pend;
        a.nct = (int)((pend - a.cbase + CB - 1) / CB);
        const int64_t nrt = (rest + CB - 1) / CB;
        k_zprod<RECT><<<(unsigned)(nrt * a.nct), 256, 0, st>>>(a);
      }
    }
    if (pend >= K) break;
    const int64_t pend2 = std::min<int64_t>(K, pend + PW);
    VMC_HIP(hipEventRecord(ctx->ev_main, st));  // panel P_p factored
    // lookahead: columns [pend, pend2), rows >= pend, reduction over P_p
    if (aux_busy) VMC_HIP(hipStreamWaitEvent(st, ctx->ev_aux, 0));
    {
      zargs a{};
      a.S = S;
      a.K = K;
      a.kb0 = p0;
      a.depth = (int)(pend - p0);
      a.rbase = pend;
      a.cbase = pend;
      a.cend = pend2;
      a.nct = (int)((pend2 - pend + CB - 1) / CB);
      a.fail = fail;
      const int64_t nrt = (K - pend + CB - 1) / CB;
      k_zprod<RECT><<<(unsigned)(nrt * a.nct), 256, 0, st>>>(a);
    }
    // the rest of the trailing matrix on the auxiliary stream
    if (pend2 < K) {
      VMC_HIP(hipStreamWaitEvent(aux, ctx->ev_main, 0));
      zargs a{};
      a.S = S;
      a.K = K;
      a.kb0 = p0;
      a.depth = (int)(pend - p0);
      a.rbase = pend2;
      a.fail = fail;
      a.nct = (int)((K - pend2 + CB - 1) / CB);
      // squares of eight tile rows where every XCD gets many of them (at least 8 each), of
      // four or single tiles below, where whole squares would leave XCDs idle
      a.sd = a.nct >= 96 ? 8 : a.nct >= 48 ? 4 : 1;
      const int64_t nsr = (a.nct + a.sd - 1) / a.sd, nsq = nsr * (nsr + 1) / 2;
      k_zprod<TRI><<<(unsigned)((nsq + 7) / 8 * 8 * a.sd * a.sd), 256, 0, aux>>>(a);
      VMC_HIP(hipEventRecord(ctx->ev_aux, aux));
      aux_busy = true;
    }
  }
  if (aux_busy) VMC_HIP(hipStreamWaitEvent(st, ctx->ev_aux, 0));
  VMC_HIP(hipGetLastError());
}

size_t chol_sync_bytes(int64_t K) { return sizeof(int) * (size_t)(2 * ((K + CB - 1) / CB) + 3); }
int chol_sync_err_index(int64_t K) { return (int)(2 * ((K + CB - 1) / CB) + 2); }

// y and x are K-vectors; x receives the solution, rhs is left unchanged;
// sync holds chol_sync_bytes(K) (its error word is set if a wait gave up)
void chol_solve(vmc_ctx* ctx, const double2* S, int64_t K, const double2* Linv, const double2* rhs, double2* y,
                double2* x, int* sync) {
  hipStream_t st = ctx->stream;
  const int nblk = (int)((K + CB - 1) / CB);
  k_zero_ints<<<1, 256, 0, st>>>(sync, 2 * nblk + 3);
  k_fwd_chain<<<(unsigned)nblk, 256, 0, st>>>(S, K, nblk, Linv, rhs, y, sync);
  k_bwd_chain<<<(unsigned)nblk, 256, 0, st>>>(S, K, nblk, Linv, y, x, sync);
  VMC_HIP(hipGetLastError());
}
