// Two-layer periodic CNN (C channels, k x k kernels, log-cosh after both
// layers, sum-pool) on an Lx x Ly torus, float64 path:
//   z1[c,p] = b1_c + sum_t W1[c,t] sigma[p + t],      a1 = logcosh(z1)
//   z2[c,p] = b2_c + sum_{c',t} W2[c,c',t] a1[c',p + t],  log psi = sum logcosh(z2)
// with p + t the periodic shift of position p by tap t = (dy, dx).
//
// Kernels:
//   k_cnn_net      log psi, O_k rows or the reverse-mode product: one
//                  work-group per sample, activations in LDS, the convolutions
//                  as matrix products on the float64 matrix cores; both layers
//                  recomputed per sample (no activations stored between calls)
//   k_cnn_forward  log psi of small networks, output by output
//   k_cnn_eloc64   local energies of the TFIM on tori of at least 2k - 1 sites a
//                  side: for a flip of site s only the k x k layer-1 positions p
//                  with p + t = s change, and only the (2k-1) x (2k-1) layer-2
//                  positions that read them, so each connected configuration
//                  costs C*C*k^4 complex multiply-adds instead of a full
//                  evaluation; 16 flips at a time as matrix products
//   k_cnn_eloc     the same without matrix products, where a sample does not fit
//                  k_cnn_eloc64's LDS or its scratch the workspace limit;
//                  smaller tori re-evaluate layer 2 in full per slot
//   k_cnn_mh64     Metropolis chains, the window's change of a proposal as a
//                  matrix product (up to 16 channels and 4 x 4 taps)
//   k_cnn_metropolis  the chains of larger networks
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "internal.h"

using namespace dev;

namespace {

struct cnn_geom {
  int Lx, Ly, N, C, k, W;
  const double2* W1;  // [C][k][k]
  const double2* b1;  // [C]
  const double2* W2;  // [C][C][k][k]
  const double2* b2;  // [C]
  // matrix-core operands of the convolutions (k_cnn_frags)
  const double2* F0;  // layer 1: [RT][KT][64]
  const double2* F1;  // layer 2 forward: [RT][kk][KS][64]
  const double2* F2;  // layer 2 backward: [RT][kk][KS][64]
  int RT, KS, KT;     // row tiles ceil(C / 16), k steps ceil(C / 4), ceil(kk / 4)
  float invLx;
};

typedef double doublex4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ doublex4 mfma64(double a, double b, doublex4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ int shift_pos(const cnn_geom& g, int p, int dy, int dx) {
  const int y = p / g.Lx, x = p - y * g.Lx;
  int yy = y + dy, xx = x + dx;
  yy %= g.Ly;
  xx %= g.Lx;
  if (yy < 0) yy += g.Ly;
  if (xx < 0) xx += g.Lx;
  return yy * g.Lx + xx;
}

__device__ __forceinline__ double sig_at(const uint64_t* s, int i) { return ((s[i >> 6] >> (i & 63)) & 1ull) ? 1.0 : -1.0; }

__device__ __forceinline__ double2 z1_at(const cnn_geom& g, const uint64_t* s, int c, int p) {
  double2 z = g.b1[c];
  for (int dy = 0; dy < g.k; ++dy)
    for (int dx = 0; dx < g.k; ++dx) {
      const double sg = sig_at(s, shift_pos(g, p, dy, dx));
      const double2 w = g.W1[(c * g.k + dy) * g.k + dx];
      z.x += sg * w.x;
      z.y += sg * w.y;
    }
  return z;
}

// layer 1 into a1[c][p] (LDS), layer 2 value at (c, p) from LDS a1
// sum_ci W2[c][ci][tap] DA[ci][w] for one (c, tap, w): w2 points at W2[c][0][tap],
// da at DA[0][w]; both advance by k*k per input channel.  Four independent
// partial sums keep several loads in flight.
__device__ __forceinline__ double2 window_tap(const double2* __restrict__ w2, const double2* __restrict__ da, int C,
                                              int kk) {
  double2 s0 = make_double2(0.0, 0.0), s1 = s0, s2 = s0, s3 = s0;
  int ci = 0;
  for (; ci + 4 <= C; ci += 4) {
    s0 = cadd(s0, cmul(w2[ci * kk], da[ci * kk]));
    s1 = cadd(s1, cmul(w2[(ci + 1) * kk], da[(ci + 1) * kk]));
    s2 = cadd(s2, cmul(w2[(ci + 2) * kk], da[(ci + 2) * kk]));
    s3 = cadd(s3, cmul(w2[(ci + 3) * kk], da[(ci + 3) * kk]));
  }
  for (; ci < C; ++ci) s0 = cadd(s0, cmul(w2[ci * kk], da[ci * kk]));
  return cadd(cadd(s0, s1), cadd(s2, s3));
}

__device__ __forceinline__ double2 z2_at(const cnn_geom& g, const double2* a1, int c, int p) {
  double2 z = g.b2[c];
  const int kk = g.k * g.k;
  for (int ci = 0; ci < g.C; ++ci)
    for (int dy = 0; dy < g.k; ++dy)
      for (int dx = 0; dx < g.k; ++dx) {
        const double2 w = g.W2[((c * g.C + ci) * g.k + dy) * g.k + dx];
        z = cadd(z, cmul(w, a1[ci * g.N + shift_pos(g, p, dy, dx)]));
      }
  (void)kk;
  return z;
}

__device__ double2 block_sum(double2 v, double2* red) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  double2 t = make_double2(0.0, 0.0);
  for (int q = 0; q < (int)(blockDim.x >> 6); ++q) t = cadd(t, red[q]);
  __syncthreads();
  return t;
}

// Weights in the operand layout of v_mfma_f64_16x16x4 (lane l holds A[l % 16][l / 16]
// of each 16 x 4 operand), one complex entry per lane, zero outside the network:
//   F0[rt][ks][l] = W1[16 rt + l % 16][tap 4 ks + l / 16]
//   F1[rt][t][ks][l] = W2[16 rt + l % 16][4 ks + l / 16][t]     (rows: output channels)
//   F2[rt][t][ks][l] = W2[4 ks + l / 16][16 rt + l % 16][t]     (rows: input channels)
// so that a wave reads an operand as one contiguous kilobyte.
__global__ void k_cnn_frags(cnn_geom g, double2* __restrict__ F, int64_t n0, int64_t n1, int64_t n) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= n) return;
  const int kk = g.k * g.k;
  const int li = (int)(e & 15), lk = (int)((e >> 4) & 3);
  double2 v = make_double2(0.0, 0.0);
  if (e < n0) {
    const int u = (int)(e >> 6), c = 16 * (u / g.KT) + li, t = 4 * (u % g.KT) + lk;
    if (c < g.C && t < kk) v = g.W1[c * kk + t];
  } else {
    const bool back = e >= n1;
    const int u = (int)((e - (back ? n1 : n0)) >> 6);
    const int ks = u % g.KS, t = (u / g.KS) % kk, row = 16 * (u / g.KS / kk) + li, col = 4 * ks + lk;
    if (row < g.C && col < g.C) v = g.W2[((back ? col * g.C + row : row * g.C + col)) * kk + t];
  }
  F[e] = v;
}

__device__ __forceinline__ void pos_yx(const cnn_geom& g, int p, int& y, int& x) {
  y = (int)(((float)p + 0.5f) * g.invLx);  // exact for p < 4096: the fraction stays 0.5 / Lx away from an integer
  x = p - y * g.Lx;
}

// Layer-1 pre-activations of row tile rt at the 16 positions of tile pt: register r
// of lane l is channel 16 rt + l / 16 + 4 r at position 16 pt + l % 16 (the
// accumulator layout of the float64 matrix cores).
__device__ __forceinline__ void z1_tile(const cnn_geom& g, const uint64_t* s, int rt, int pt, int lane, doublex4& re,
                                        doublex4& im) {
  const int li = lane & 15, lk = lane >> 4, kk = g.k * g.k;
  int y, x;
  pos_yx(g, min(pt * 16 + li, g.N - 1), y, x);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const double2 b = g.b1[min(rt * 16 + lk + 4 * r, g.C - 1)];
    re[r] = b.x;
    im[r] = b.y;
  }
  for (int ks = 0; ks < g.KT; ++ks) {
    const int t = min(4 * ks + lk, kk - 1), dy = t / g.k, dx = t - dy * g.k;
    int yy = y + dy, xx = x + dx;
    yy -= yy >= g.Ly ? g.Ly : 0;
    xx -= xx >= g.Lx ? g.Lx : 0;
    const double sg = sig_at(s, yy * g.Lx + xx);
    const double2 w = g.F0[(size_t)(rt * g.KT + ks) * 64 + lane];  // 0 past the last tap
    re = mfma64(w.x, sg, re);
    im = mfma64(w.y, sg, im);
  }
}

// NP tiles of 16 positions (tiles pt0 .. pt0 + NP - 1) of the layer-2 convolution of
// X (LDS, [C][ld]) with the operands F: acc += sum_{t, c'} F[rt][t](row, c') X[c'][p +- t]
// (SGN = 1: p + t, the forward convolution; SGN = -1: p - t, its transpose).
template <int NP, int SGN>
__device__ __forceinline__ void conv_tiles(const cnn_geom& g, const double2* __restrict__ F, const double2* X, int ld,
                                           int rt, int pt0, int lane, doublex4 (&re)[NP], doublex4 (&im)[NP]) {
  const int li = lane & 15, lk = lane >> 4, kk = g.k * g.k;
  int py[NP], px[NP];
#pragma unroll
  for (int j = 0; j < NP; ++j) pos_yx(g, min((pt0 + j) * 16 + li, g.N - 1), py[j], px[j]);
  const double2* Fr = F + (size_t)rt * kk * g.KS * 64 + lane;
  const int last = kk * g.KS - 1;
  double2 a = Fr[0];
  int u = 0;
  for (int dy = 0; dy < g.k; ++dy)
    for (int dx = 0; dx < g.k; ++dx) {
      int q[NP];
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        int yy = py[j] + SGN * dy, xx = px[j] + SGN * dx;
        if (SGN > 0) {
          yy -= yy >= g.Ly ? g.Ly : 0;
          xx -= xx >= g.Lx ? g.Lx : 0;
        } else {
          yy += yy < 0 ? g.Ly : 0;
          xx += xx < 0 ? g.Lx : 0;
        }
        q[j] = yy * g.Lx + xx;
      }
      for (int ks = 0; ks < g.KS; ++ks, ++u) {
        const double2 an = Fr[(size_t)min(u + 1, last) * 64];  // the next operand in flight
        const double2* row = X + min(4 * ks + lk, g.C - 1) * ld;  // F is 0 past the last channel
        double2 b[NP];
#pragma unroll
        for (int j = 0; j < NP; ++j) b[j] = row[q[j]];
        const double na = -a.y;
#pragma unroll
        for (int j = 0; j < NP; ++j) {
          re[j] = mfma64(a.x, b[j].x, re[j]);
          im[j] = mfma64(a.x, b[j].y, im[j]);
        }
#pragma unroll
        for (int j = 0; j < NP; ++j) {
          re[j] = mfma64(na, b[j].y, re[j]);
          im[j] = mfma64(a.y, b[j].x, im[j]);
        }
        a = an;
      }
    }
}

// log psi, a work-group per sample and a thread per output at a time, for networks that would
// fill little of the matrix cores' operands.  LDS: a1 [C][N], four partial sums.
// Bound: latency, and index arithmetic with every term.
__global__ __launch_bounds__(256) void k_cnn_forward(cnn_geom g, const uint64_t* __restrict__ s, int64_t B,
                                                     double2* __restrict__ logpsi) {
  extern __shared__ double2 sm[];
  const int64_t b = blockIdx.x;
  if (b >= B) return;
  const int CN = g.C * g.N;
  double2* a1 = sm;
  double2* red = sm + CN;
  const uint64_t* sb = s + b * g.W;
  for (int e = threadIdx.x; e < CN; e += 256) a1[e] = clogcosh_pv(z1_at(g, sb, e / g.N, e % g.N));
  __syncthreads();
  double2 acc = make_double2(0.0, 0.0);
  for (int e = threadIdx.x; e < CN; e += 256) acc = cadd(acc, clogcosh(z2_at(g, a1, e / g.N, e % g.N)));
  acc = block_sum(acc, red);
  if (threadIdx.x == 0) logpsi[b] = acc;
}

constexpr int NET_NT = 512;  // threads of a sample's work-group, at most (net_threads)
constexpr int NP = 2;  // tiles of a wave that share an operand
enum { NET_LOGPSI = 0, NET_ROWS = 1, NET_VJP = 2 };

// One sample per work-group, every contraction of the network as float64 matrix
// products (16 x 16 blocks, four real products per complex term):
//   layer 1       z1[c][p]        rows c, columns p, reduction over taps
//   layer 2       z2[c][p]        rows c, columns p, reduction over (tap, c')
//   dW2[c][c',t] = sum_p g2[c][p] a1[c'][p + t]     rows c, columns (c', t), reduction over p
//   back[c'][p]  = sum_{c,t} W2[c][c'][t] g2[c][p - t]   (the forward product, transposed)
//   dW1[c][t]    = sum_p g1[c][p] sigma[p + t]      rows c, columns t, reduction over p
// with a1 = logcosh(z1), g2 = tanh(z2), g1 = back tanh(z1).  LDS: A [C][N + 1]
// (a1, later g1), G2 [C][N + 1] (g2, later partial sums of dW1); the odd row
// length spreads the rows over the banks where lanes run over channels.
// Rows O_k = [W1 (C k k), b1 (C), W2 (C C k k), b2 (C)].  MODE NET_ROWS writes
// O_k(s_b) to row b of O; NET_VJP accumulates g_b conj(O_k(s_b)) over the group's
// samples x, x + gridDim.x, ... into row x of part, each entry by the one thread
// that forms it; NET_LOGPSI stops after layer 2.
//
// Bound: the float64 matrix cores (12 C^2 k^2 N real multiply-adds for the three
// layer-2 products: 83 us a sample and compute unit at C = 16, k = 4, N = 256 at
// the full rate, 0.33 of the 0.60 ms below); the rest is the transcendental
// functions of the two activations and the operand latency of two groups a compute unit
// (16 waves a group with one tile each: 0.61 ms).  Log psi is held to 80 registers, which leave
// three groups a compute unit.  The loops over
// taps and positions per output that this replaces spent their time on index
// arithmetic and serial sums.
// 1 024 samples, 16 x 16, C = 16, k = 4: log psi 1.53 -> 0.23 ms, O_k (complex64)
// 7.92 -> 0.60 ms, reverse-mode product 7.86 -> 0.67 ms.
template <int MODE, int NT, typename OutT>
__global__ __launch_bounds__(NT, MODE == NET_LOGPSI ? 6 : 2) void k_cnn_net(
    cnn_geom g, const uint64_t* __restrict__ s, int64_t B, int64_t K, OutT* __restrict__ O,
    const double2* __restrict__ gv, double2* __restrict__ part, double2* __restrict__ logpsi) {
  constexpr int NW = NT / 64;
  extern __shared__ double2 sm[];
  __shared__ double2 red[NW];
  const int C = g.C, N = g.N, ld = N + 1, kk = g.k * g.k;
  double2* A = sm;
  double2* G2 = sm + C * ld;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int PT = (N + 15) / 16, PP = (PT + NP - 1) / NP;  // position tiles, groups of them
  const int off_b1 = C * kk, off_W2 = off_b1 + C, off_b2 = off_W2 + C * C * kk;
  for (int64_t b = blockIdx.x; b < B; b += gridDim.x) {
    const uint64_t* sb = s + b * g.W;
    const bool first = b == (int64_t)blockIdx.x;
    const double2 gb = MODE == NET_VJP ? gv[b] : make_double2(0.0, 0.0);
    auto put = [&](int64_t k, double2 v) {
      if constexpr (MODE == NET_VJP) {
        const double2 t = cmul(gb, cconj(v));
        double2* q = part + (int64_t)blockIdx.x * K + k;
        *q = first ? t : cadd(*q, t);
      } else if constexpr (MODE == NET_ROWS) {
        OutT* row = O + b * K;
        if constexpr (sizeof(OutT) == sizeof(double2))
          row[k] = v;
        else
          row[k] = make_float2((float)v.x, (float)v.y);
      }
    };
    __syncthreads();  // the previous sample's last LDS reads are done
    for (int u = wave; u < g.RT * PT; u += NW) {
      const int rt = u / PT, pt = u - rt * PT;
      doublex4 re, im;
      z1_tile(g, sb, rt, pt, lane, re, im);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int c = rt * 16 + lk + 4 * r, p = pt * 16 + li;
        if (c < C && p < N) A[c * ld + p] = clogcosh_pv(make_double2(re[r], im[r]));
      }
    }
    __syncthreads();
    double2 lp = make_double2(0.0, 0.0);
    for (int u = wave; u < g.RT * PP; u += NW) {
      const int rt = u / PP, pt = NP * (u - rt * PP);
      doublex4 re[NP], im[NP];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double2 b2 = g.b2[min(rt * 16 + lk + 4 * r, C - 1)];
        for (int j = 0; j < NP; ++j) {
          re[j][r] = b2.x;
          im[j][r] = b2.y;
        }
      }
      conv_tiles<NP, 1>(g, g.F1, A, ld, rt, pt, lane, re, im);
#pragma unroll
      for (int j = 0; j < NP; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int c = rt * 16 + lk + 4 * r, p = (pt + j) * 16 + li;
          if (c < C && p < N) {
            const double2 z = make_double2(re[j][r], im[j][r]);
            if constexpr (MODE == NET_LOGPSI)
              lp = cadd(lp, clogcosh(z));
            else
              G2[c * ld + p] = ctanh(z);
          }
        }
    }
    if constexpr (MODE == NET_LOGPSI) {
      lp = wave_sum(lp);
      if (lane == 0) red[wave] = lp;
      __syncthreads();
      if (tid == 0) {
        double2 t = make_double2(0.0, 0.0);
        for (int w = 0; w < NW; ++w) t = cadd(t, red[w]);
        logpsi[b] = t;
      }
      continue;
    }
    __syncthreads();
    // dW2: two tiles of 16 columns (c', t) share the rows g2
    const int CT = (C * kk + 15) / 16, CP = (CT + NP - 1) / NP;
    for (int u = wave; u < g.RT * CP; u += NW) {
      const int rt = u / CP, ct = NP * (u - rt * CP);
      const double2* arow = G2 + min(rt * 16 + li, C - 1) * ld;
      const double2* brow[NP];
      int dy[NP], dx[NP];
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        const int n = min((ct + j) * 16 + li, C * kk - 1), ci = n / kk, t = n - ci * kk;
        brow[j] = A + ci * ld;
        dy[j] = t / g.k;
        dx[j] = t - dy[j] * g.k;
      }
      doublex4 re[NP], im[NP];
      for (int j = 0; j < NP; ++j) re[j] = im[j] = doublex4{0.0, 0.0, 0.0, 0.0};
      for (int p0 = 0; p0 < N; p0 += 4) {
        const int p = min(p0 + lk, N - 1);
        int y, x;
        pos_yx(g, p, y, x);
        double2 a = arow[p];
        if (p0 + lk >= N) a = make_double2(0.0, 0.0);
        double2 bv[NP];
#pragma unroll
        for (int j = 0; j < NP; ++j) {
          int yy = y + dy[j], xx = x + dx[j];
          yy -= yy >= g.Ly ? g.Ly : 0;
          xx -= xx >= g.Lx ? g.Lx : 0;
          bv[j] = brow[j][yy * g.Lx + xx];
        }
        const double na = -a.y;
#pragma unroll
        for (int j = 0; j < NP; ++j) {
          re[j] = mfma64(a.x, bv[j].x, re[j]);
          im[j] = mfma64(a.x, bv[j].y, im[j]);
        }
#pragma unroll
        for (int j = 0; j < NP; ++j) {
          re[j] = mfma64(na, bv[j].y, re[j]);
          im[j] = mfma64(a.y, bv[j].x, im[j]);
        }
      }
#pragma unroll
      for (int j = 0; j < NP; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int c = rt * 16 + lk + 4 * r, n = (ct + j) * 16 + li;
          if (c < C && n < C * kk) put(off_W2 + (int64_t)c * C * kk + n, make_double2(re[j][r], im[j][r]));
        }
    }
    for (int c = wave; c < C; c += NW) {
      double2 acc = make_double2(0.0, 0.0);
      for (int p = lane; p < N; p += 64) acc = cadd(acc, G2[c * ld + p]);
      acc = wave_sum(acc);
      if (lane == 0) put(off_b2 + c, acc);
    }
    __syncthreads();  // a1 is no longer read
    // g1 = tanh(z1) d log psi / d a1 -> A
    for (int u = wave; u < g.RT * PP; u += NW) {
      const int rt = u / PP, pt = NP * (u - rt * PP);
      doublex4 re[NP], im[NP];
      for (int j = 0; j < NP; ++j) re[j] = im[j] = doublex4{0.0, 0.0, 0.0, 0.0};
      conv_tiles<NP, -1>(g, g.F2, G2, ld, rt, pt, lane, re, im);
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        if (pt + j >= PT) break;
        doublex4 zr, zi;
        z1_tile(g, sb, rt, pt + j, lane, zr, zi);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int c = rt * 16 + lk + 4 * r, p = (pt + j) * 16 + li;
          if (c < C && p < N)
            A[c * ld + p] = cmul(make_double2(re[j][r], im[j][r]), ctanh(make_double2(zr[r], zi[r])));
        }
      }
    }
    __syncthreads();
    // dW1: tiles of (16 channels, 16 taps); the positions split over ns parts (as many as
    // the waves and the partial sums in G2 allow), added in a fixed order
    const int TT = (kk + 15) / 16, nt = g.RT * TT;
    int ns = 1;
    while (ns < NW && 2 * ns * nt * 256 <= C * ld) ns *= 2;
    const int per = ((N + ns - 1) / ns + 3) / 4 * 4;
    for (int u = wave; u < nt * ns; u += NW) {
      const int tile = u / ns, z = u - tile * ns, rt = tile / TT, t0 = 16 * (tile - rt * TT);
      const double2* arow = A + min(rt * 16 + li, C - 1) * ld;
      const int t = min(t0 + li, kk - 1), dy = t / g.k, dx = t - dy * g.k;
      doublex4 re = doublex4{0.0, 0.0, 0.0, 0.0}, im = re;
      const int pe = min(N, (z + 1) * per);
      for (int p0 = z * per; p0 < pe; p0 += 4) {
        const int p = min(p0 + lk, N - 1);
        int y, x;
        pos_yx(g, p, y, x);
        y += dy;
        x += dx;
        y -= y >= g.Ly ? g.Ly : 0;
        x -= x >= g.Lx ? g.Lx : 0;
        const double sg = p0 + lk < pe ? sig_at(sb, y * g.Lx + x) : 0.0;
        const double2 a = arow[p];
        re = mfma64(a.x, sg, re);
        im = mfma64(a.y, sg, im);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = lk + 4 * r, c = rt * 16 + row;
        if (ns > 1)
          G2[(tile * ns + z) * 256 + row * 16 + li] = make_double2(re[r], im[r]);
        else if (c < C && t0 + li < kk)
          put(c * kk + t0 + li, make_double2(re[r], im[r]));
      }
    }
    for (int c = wave; c < C; c += NW) {
      double2 acc = make_double2(0.0, 0.0);
      for (int p = lane; p < N; p += 64) acc = cadd(acc, A[c * ld + p]);
      acc = wave_sum(acc);
      if (lane == 0) put(off_b1 + c, acc);
    }
    if (ns > 1) {
      __syncthreads();
      for (int e = tid; e < nt * 256; e += NT) {
        const int tile = e >> 8, rt = tile / TT, c = rt * 16 + ((e >> 4) & 15), t = 16 * (tile - rt * TT) + (e & 15);
        if (c < C && t < kk) {
          double2 acc = make_double2(0.0, 0.0);
          for (int z = 0; z < ns; ++z) acc = cadd(acc, G2[(tile * ns + z) * 256 + (e & 255)]);
          put(c * kk + t, acc);
        }
      }
    }
  }
}

constexpr int EL_NT = 1024;
constexpr int EL_NW = EL_NT / 64;
constexpr int EL_F = 16;  // flips per pass: the columns of one matrix-core operand

// 1 + e^{-2 z~} with z~ = +-z, Re z~ >= 0 (cosh z = e^{z~} (1 + e^{-2 z~}) / 2); zt receives z~
__device__ __forceinline__ double2 cosh_factor(double2 z, double2& zt) {
  zt = z.x < 0.0 ? make_double2(-z.x, -z.y) : z;
  const double e = m64::fexp_neg0(2.0 * zt.x);
  double s, c;
  m64::fsincos(-2.0 * zt.y, &s, &c);
  return make_double2(fma(e, c, 1.0), e * s);
}

// TFIM local energies on tori of at least 2k - 1 sites a side, matrix-core form.
// For a flip of site f the layer-1 changes dA[c'][t1] sit at the positions f - t1 and
// the layer-2 changes at f - e, e = t1 + t2:
//   dZ[c][e] = sum_{t1 + t2 = e} sum_{c'} W2[c][c'][t2] dA[c'][t1].
// A pass takes EL_F = 16 consecutive sites as the columns of the products: per window
// offset e the rows are 16 output channels and the reduction runs over the pairs
// (t1, t2) and c', so no entry of a product is padding (C a multiple of 16) and a
// column's window is summed without leaving its lanes.  The (row tile, e) units are
// shared out over the waves by cost on the host.  Each lane then multiplies
//   cosh(z2 + dZ) / cosh(z2) = e^{z~' - z~} (1 + e^{-2 z~'}) / (1 + e^{-2 z~})
// over its outputs as a product with a separate exponent and one logarithm per pass,
// instead of a logarithm and an arctangent per output.
// LDS: Z2 [C][N + 1], dA [C][kk][16] (before the passes: a1 [C][N + 1]); z1, a1 and
// 1 / (1 + e^{-2 z~}) of the work-group's sample in global scratch.
//
// Bound: the float64 matrix cores and the float64 vector work of the factors, which
// hardly overlap: the matrix pipe is busy 51% of the cycles (4 C^2 k^4 N real
// multiply-adds a sample, 443 us a compute unit at C = 16, k = 4, N = 256), vector
// instructions issue in 40% (counters).  512 samples of that network: 25.2 -> 1.81 ms (with
// 8 instead of 16 waves a group 6% more).
template <int KSC>
__global__ __launch_bounds__(EL_NT, 4) void k_cnn_eloc64(cnn_geom g, const uint64_t* __restrict__ s, int64_t B,
                                                         int nsplit, double J, double h,
                                                         const int2* __restrict__ bonds, int n_bonds,
                                                         const int* __restrict__ units, double2* __restrict__ scr,
                                                         double2* __restrict__ eloc) {
  extern __shared__ double2 sm[];
  __shared__ double2 red[EL_NW][EL_F];
  __shared__ int nal_s[EL_NW];
  const int C = g.C, N = g.N, ld = N + 1, k = g.k, kk = k * k, win = 2 * k - 1;
  const int CN = C * N;
  const int KS = KSC ? KSC : g.KS;
  double2* Z2 = sm;
  double2* DA = sm + C * ld;
  double2* z1g = scr + (size_t)blockIdx.x * 3 * CN;
  double2* a1g = z1g + CN;
  double2* iqg = a1g + CN;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const int PT = (N + 15) / 16, PP = (PT + 1) / 2;
  const int npass = (N + EL_F - 1) / EL_F;
  const int u0 = units[wave], u1 = units[wave + 1];
  for (int64_t item = blockIdx.x; item < B * nsplit; item += gridDim.x) {
    const int64_t b = item / nsplit;
    const int sp = (int)(item - b * nsplit);
    const uint64_t* sb = s + b * g.W;
    __syncthreads();  // the previous sample's LDS and scratch reads are done
    for (int u = wave; u < g.RT * PT; u += EL_NW) {
      const int rt = u / PT, pt = u - rt * PT;
      doublex4 re, im;
      z1_tile(g, sb, rt, pt, lane, re, im);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int c = rt * 16 + lk + 4 * r, p = pt * 16 + li;
        if (c < C && p < N) {
          const double2 z = make_double2(re[r], im[r]), a = clogcosh_pv(z);
          DA[c * ld + p] = a;
          z1g[c * N + p] = z;
          a1g[c * N + p] = a;
        }
      }
    }
    __syncthreads();
    for (int u = wave; u < g.RT * PP; u += EL_NW) {
      const int rt = u / PP, pt = NP * (u - rt * PP);
      doublex4 re[NP], im[NP];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double2 b2 = g.b2[min(rt * 16 + lk + 4 * r, C - 1)];
        for (int j = 0; j < NP; ++j) {
          re[j][r] = b2.x;
          im[j][r] = b2.y;
        }
      }
      conv_tiles<NP, 1>(g, g.F1, DA, ld, rt, pt, lane, re, im);
#pragma unroll
      for (int j = 0; j < NP; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int c = rt * 16 + lk + 4 * r, p = (pt + j) * 16 + li;
          if (c < C && p < N) {
            const double2 z = make_double2(re[j][r], im[j][r]);
            double2 zt;
            const double2 q = cosh_factor(z, zt);
            Z2[c * ld + p] = z;
            iqg[c * N + p] = cdiv(make_double2(1.0, 0.0), q);
          }
        }
    }
    int n_al = 0;
    if (sp == 0)
      for (int q = tid; q < n_bonds; q += EL_NT) n_al += sig_at(sb, bonds[q].x) == sig_at(sb, bonds[q].y);
    n_al = wave_isum_uniform(n_al);
    if (lane == 0) nal_s[wave] = n_al;
    __syncthreads();
    double2 acc = make_double2(0.0, 0.0);  // threads 0..15: their column's sites
    for (int ps = sp; ps < npass; ps += nsplit) {
      // dA[c][t1][column]
      for (int e = tid; e < C * kk * EL_F; e += EL_NT) {
        const int f = min(ps * EL_F + (e & (EL_F - 1)), N - 1), r = e / EL_F, c = r / kk, t = r - c * kk;
        const int dy = t / k, dx = t - dy * k;
        int y, x;
        pos_yx(g, f, y, x);
        y -= dy;
        x -= dx;
        y += y < 0 ? g.Ly : 0;
        x += x < 0 ? g.Lx : 0;
        const int p = y * g.Lx + x;
        const double ds = -2.0 * sig_at(sb, f);
        const double2 z = z1g[c * N + p], w = g.W1[c * kk + t];
        DA[e] = csub(clogcosh_pv(make_double2(fma(ds, w.x, z.x), fma(ds, w.y, z.y))), a1g[c * N + p]);
      }
      __syncthreads();
      int fy, fx;
      pos_yx(g, min(ps * EL_F + li, N - 1), fy, fx);
      double2 P = make_double2(1.0, 0.0), lin = make_double2(0.0, 0.0);
      int ex2 = 0;
      for (int uu = u0; uu < u1; ++uu) {
        const int un = __builtin_amdgcn_readfirstlane(units[uu]);
        const int rt = un >> 16, ey = (un >> 8) & 255, ex = un & 255;
        int qy = fy - ey, qx = fx - ex;
        qy += qy < 0 ? g.Ly : 0;
        qx += qx < 0 ? g.Lx : 0;
        const int q = qy * g.Lx + qx;
        double2 iq[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) iq[r] = iqg[min(rt * 16 + lk + 4 * r, C - 1) * N + q];
        doublex4 re0 = doublex4{0.0, 0.0, 0.0, 0.0}, re1 = re0, im0 = re0, im1 = re0;
        const int ylo = max(0, ey - k + 1), yhi = min(k - 1, ey), xlo = max(0, ex - k + 1), xhi = min(k - 1, ex);
        const double2* Fr = g.F1 + (size_t)rt * kk * KS * 64 + lane;
        for (int y2 = ylo; y2 <= yhi; ++y2)
          for (int x2 = xlo; x2 <= xhi; ++x2) {
            const double2* fa = Fr + (size_t)(y2 * k + x2) * KS * 64;
            const double2* db = DA + ((ey - y2) * k + ex - x2) * EL_F + li;
            auto step = [&](double2 a, double2 d) {
              re0 = mfma64(a.x, d.x, re0);
              im0 = mfma64(a.x, d.y, im0);
              re1 = mfma64(-a.y, d.y, re1);
              im1 = mfma64(a.y, d.x, im1);
            };
            if constexpr (KSC > 0) {
              double2 a[KSC], d[KSC];
#pragma unroll
              for (int ks = 0; ks < KSC; ++ks) {
                a[ks] = fa[ks * 64];
                d[ks] = db[min(4 * ks + lk, C - 1) * kk * EL_F];
              }
#pragma unroll
              for (int ks = 0; ks < KSC; ++ks) step(a[ks], d[ks]);
            } else {
              for (int ks = 0; ks < KS; ++ks) step(fa[ks * 64], db[min(4 * ks + lk, C - 1) * kk * EL_F]);
            }
          }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int c = rt * 16 + lk + 4 * r;
          if (c >= C) continue;
          const double2 z = Z2[c * ld + q], dz = make_double2(re0[r] + re1[r], im0[r] + im1[r]);
          double2 zt;
          const double2 f = cmul(cosh_factor(cadd(z, dz), zt), iq[r]);
          const double sg = z.x < 0.0 ? -1.0 : 1.0;
          lin = cadd(lin, csub(zt, cscale(z, sg)));
          P = cmul(P, f);
        }
        const int e2 = __builtin_amdgcn_frexp_exp(fmax(fabs(P.x), fabs(P.y)));
        P = make_double2(ldexp(P.x, -e2), ldexp(P.y, -e2));
        ex2 += e2;
      }
      double2 L = clog(P);
      L = make_double2(lin.x + (L.x + 0.69314718055994530942 * (double)ex2), lin.y + L.y);
      L.x += __shfl_xor(L.x, 16, 64);
      L.y += __shfl_xor(L.y, 16, 64);
      L.x += __shfl_xor(L.x, 32, 64);
      L.y += __shfl_xor(L.y, 32, 64);
      if (lk == 0) red[wave][li] = L;
      __syncthreads();
      if (tid < EL_F && ps * EL_F + tid < N) {
        double2 t = make_double2(0.0, 0.0);
        for (int w = 0; w < EL_NW; ++w) t = cadd(t, red[w][tid]);
        acc = cadd(acc, cscale(cexp(t), -h));
      }
    }
    if (tid < 64) {  // lanes 16 .. 63 hold 0
      acc = wave_sum(acc);
      if (tid == 0) {
        if (sp == 0) {
          int nal = 0;
          for (int w = 0; w < EL_NW; ++w) nal += nal_s[w];
          acc.x += -J * (double)(nal - (n_bonds - nal));
        }
        eloc[item] = acc;
      }
    }
  }
}

// eloc[b] = sum of the nsplit parts of sample b, in order
__global__ void k_cnn_eloc_add(const double2* __restrict__ part, int64_t B, int nsplit, double2* __restrict__ eloc) {
  const int64_t b = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (b >= B) return;
  double2 acc = part[b * nsplit];
  for (int q = 1; q < nsplit; ++q) acc = cadd(acc, part[b * nsplit + q]);
  eloc[b] = acc;
}

// TFIM local energies.  LDS: z2 [C][N], lc2 = logcosh(z2) [C][N], da1 [C][k*k]
// (the changed layer-1 values of the current flip), sigma words, reduction.
__global__ __launch_bounds__(256) void k_cnn_eloc(cnn_geom g, const uint64_t* __restrict__ s, int64_t B, double J,
                                                  double h, const int2* __restrict__ bonds, int n_bonds,
                                                  double2* __restrict__ eloc, double2* __restrict__ a1_scratch) {
  extern __shared__ double2 sm[];
  const int CN = g.C * g.N, kk = g.k * g.k;
  double2* Z2 = sm;
  double2* LC2 = sm + CN;
  double2* DA = sm + 2 * CN;         // [C][kk]
  double2* red = DA + g.C * kk;      // [4]
  const int64_t b = blockIdx.x;
  if (b >= B) return;
  const uint64_t* sb = s + b * g.W;
  double2* a1 = a1_scratch + b * CN;  // global scratch for the full layer 1 of this sample
  const int tid = threadIdx.x;
  for (int e = tid; e < CN; e += 256) a1[e] = clogcosh_pv(z1_at(g, sb, e / g.N, e % g.N));
  __syncthreads();
  for (int e = tid; e < CN; e += 256) {
    const double2 z = z2_at(g, a1, e / g.N, e % g.N);
    Z2[e] = z;
    LC2[e] = clogcosh(z);
  }
  // diagonal element
  int n_al = 0;
  for (int q = tid; q < n_bonds; q += 256) n_al += sig_at(sb, bonds[q].x) == sig_at(sb, bonds[q].y);
  __syncthreads();
  double2 tot = block_sum(make_double2((double)n_al, 0.0), red);
  const int nal = (int)tot.x;
  const double diag = -J * (double)(nal - (n_bonds - nal));
  double2 acc = make_double2(0.0, 0.0);
  const int win = 2 * g.k - 1;
  const bool incremental = g.Lx >= win && g.Ly >= win;
  if (h != 0.0) {
    for (int site = 0; site < g.N; ++site) {
      const double ds = -2.0 * sig_at(sb, site);
      const int Ys = site / g.Lx, Xs = site % g.Lx;
      // changed layer-1 values: positions p = site - (dy, dx)
      for (int e = tid; e < g.C * kk; e += 256) {
        const int c = e / kk, t = e % kk, dy = t / g.k, dx = t % g.k;
        const int p = shift_pos(g, site, -dy, -dx);
        const double2 z = z1_at(g, sb, c, p);
        const double2 w = g.W1[(c * g.k + dy) * g.k + dx];
        const double2 zn = make_double2(z.x + ds * w.x, z.y + ds * w.y);
        DA[e] = csub(clogcosh_pv(zn), clogcosh_pv(z));
      }
      __syncthreads();
      double2 part = make_double2(0.0, 0.0);
      if (incremental) {
        // affected layer-2 outputs: q = site - (ey, ex), 0 <= ey, ex < 2k - 1
        for (int e = tid; e < g.C * win * win; e += 256) {
          const int c = e / (win * win), r = e % (win * win), ey = r / win, ex = r % win;
          double2 dz = make_double2(0.0, 0.0);
          for (int dy1 = max(0, ey - g.k + 1); dy1 <= min(g.k - 1, ey); ++dy1)
            for (int dx1 = max(0, ex - g.k + 1); dx1 <= min(g.k - 1, ex); ++dx1) {
              const int dy2 = ey - dy1, dx2 = ex - dx1;  // tap from q to the changed position
              dz = cadd(dz, window_tap(g.W2 + (c * g.C * g.k + dy2) * g.k + dx2, DA + dy1 * g.k + dx1, g.C, kk));
            }
          int qy = Ys - ey, qx = Xs - ex;
          if (qy < 0) qy += g.Ly;
          if (qx < 0) qx += g.Lx;
          const int qi = c * g.N + qy * g.Lx + qx;
          part = cadd(part, csub(clogcosh(cadd(Z2[qi], dz)), LC2[qi]));
        }
      } else {
        // small torus: re-evaluate layer 2 from the updated layer 1
        for (int e = tid; e < CN; e += 256) {
          const int c = e / g.N, q = e % g.N;
          double2 dz = make_double2(0.0, 0.0);
          for (int ci = 0; ci < g.C; ++ci)
            for (int dy = 0; dy < g.k; ++dy)
              for (int dx = 0; dx < g.k; ++dx) {
                const int p = shift_pos(g, q, dy, dx);
                // the flip changes a1[ci][p] through every tap that lands on the site
                const double2 zo = z1_at(g, sb, ci, p);
                double2 zn = zo;
                for (int ty = 0; ty < g.k; ++ty)
                  for (int tx = 0; tx < g.k; ++tx)
                    if (shift_pos(g, p, ty, tx) == site) {
                      const double2 w = g.W1[(ci * g.k + ty) * g.k + tx];
                      zn.x += ds * w.x;
                      zn.y += ds * w.y;
                    }
                if (zn.x != zo.x || zn.y != zo.y)
                  dz = cadd(dz, cmul(g.W2[((c * g.C + ci) * g.k + dy) * g.k + dx], csub(clogcosh_pv(zn), a1[ci * g.N + p])));
              }
          part = cadd(part, csub(clogcosh(cadd(Z2[e], dz)), LC2[e]));
        }
      }
      const double2 dl = block_sum(part, red);
      acc = cadd(acc, cscale(cexp(dl), -h));
      __syncthreads();
    }
  }
  if (tid == 0) eloc[b] = make_double2(acc.x + diag, acc.y);
}

// Metropolis chains for the CNN (single-spin flips; the randomness of
// sampler.hip): one work-group per chain, z2 and Re log cosh(z2) of the current
// configuration in LDS, layer 1 of the chain in global scratch.  A proposal
// evaluates Re(log psi(s') - log psi(s)) on the (2k-1) x (2k-1) window only;
// on acceptance the window of z2 is updated in place.
__global__ __launch_bounds__(256) void k_cnn_metropolis(cnn_geom g, int n_chains, uint64_t* __restrict__ bits,
                                                        uint2 key, uint64_t t0, int init, int64_t therm_steps,
                                                        int64_t n_record, int sweep, uint64_t* __restrict__ s_out,
                                                        double2* __restrict__ logpsi_out,
                                                        unsigned long long* __restrict__ acc,
                                                        double2* __restrict__ a1_scratch) {
  extern __shared__ double2 sm[];
  const int CN = g.C * g.N, kk = g.k * g.k, win = 2 * g.k - 1;
  double2* Z2 = sm;                        // [C][N]
  double* RL = (double*)(sm + CN);         // [C][N] Re logcosh(z2)
  double2* DA = sm + CN + (CN + 1) / 2;    // [C][kk]
  double2* red = DA + g.C * kk;            // [4]
  uint64_t* cb = (uint64_t*)(red + 4);     // [W]
  const int c = blockIdx.x;
  if (c >= n_chains) return;
  const int tid = threadIdx.x;
  double2* a1 = a1_scratch + (int64_t)c * CN;
  if (init) {
    if (tid == 0)
      for (int w = 0; w < g.W; ++w) {
        uint4 y = philox(make_uint4((uint32_t)c, (uint32_t)(w >> 1), 0u, 2u), key);
        uint64_t word = (w & 1) ? ((uint64_t)y.z | ((uint64_t)y.w << 32)) : ((uint64_t)y.x | ((uint64_t)y.y << 32));
        const int rem = g.N - 64 * w;
        if (rem < 64) word &= (1ull << rem) - 1ull;
        cb[w] = word;
      }
  } else {
    for (int w = tid; w < g.W; w += 256) cb[w] = bits[(int64_t)c * g.W + w];
  }
  __syncthreads();
  for (int e = tid; e < CN; e += 256) a1[e] = clogcosh_pv(z1_at(g, cb, e / g.N, e % g.N));
  __syncthreads();
  for (int e = tid; e < CN; e += 256) {
    const double2 z = z2_at(g, a1, e / g.N, e % g.N);
    Z2[e] = z;
    RL[e] = clogcosh(z).x;
  }
  __syncthreads();
  unsigned long long accepted = 0;
  const int64_t total = therm_steps + n_record * sweep;
  constexpr int MAXOUT = 8;  // window outputs per thread (C (2k-1)^2 <= 2048)
  for (int64_t step = 0; step < total; ++step) {
    const uint64_t t = t0 + (uint64_t)step;
    const uint4 x = philox(make_uint4((uint32_t)c, (uint32_t)t, (uint32_t)(t >> 32), 0u), key);
    const int site = (int)to_index(x.x, (uint32_t)g.N);
    const double u = to_uniform(x.y, x.z);
    const double ds = -2.0 * sig_at(cb, site);
    const int Ys = site / g.Lx, Xs = site % g.Lx;
    for (int e = tid; e < g.C * kk; e += 256) {
      const int ch = e / kk, tp = e % kk, dy = tp / g.k, dx = tp % g.k;
      const int p = shift_pos(g, site, -dy, -dx);
      const double2 z = z1_at(g, cb, ch, p);
      const double2 w = g.W1[(ch * g.k + dy) * g.k + dx];
      DA[e] = csub(clogcosh_pv(make_double2(z.x + ds * w.x, z.y + ds * w.y)), a1[ch * g.N + p]);
    }
    __syncthreads();
    double2 dzs[MAXOUT];
    double part = 0.0;
#pragma unroll
    for (int q = 0; q < MAXOUT; ++q) {
      const int e = tid + 256 * q;
      dzs[q] = make_double2(0.0, 0.0);
      if (e >= g.C * win * win) continue;
      const int ch = e / (win * win), r = e % (win * win), ey = r / win, ex = r % win;
      double2 dz = make_double2(0.0, 0.0);
      for (int dy1 = max(0, ey - g.k + 1); dy1 <= min(g.k - 1, ey); ++dy1)
        for (int dx1 = max(0, ex - g.k + 1); dx1 <= min(g.k - 1, ex); ++dx1)
          dz = cadd(dz, window_tap(g.W2 + (ch * g.C * g.k + ey - dy1) * g.k + ex - dx1, DA + dy1 * g.k + dx1, g.C, kk));
      dzs[q] = dz;
      int qy = Ys - ey, qx = Xs - ex;
      if (qy < 0) qy += g.Ly;
      if (qx < 0) qx += g.Lx;
      const int qi = ch * g.N + qy * g.Lx + qx;
      part += clogcosh(cadd(Z2[qi], dz)).x - RL[qi];
    }
    const double r = 2.0 * block_sum(make_double2(part, 0.0), red).x;
    const bool accept = (r >= 0.0) || (u < exp(r));
    if (accept) {
      ++accepted;
#pragma unroll
      for (int q = 0; q < MAXOUT; ++q) {
        const int e = tid + 256 * q;
        if (e >= g.C * win * win) continue;
        const int ch = e / (win * win), rr = e % (win * win), ey = rr / win, ex = rr % win;
        int qy = Ys - ey, qx = Xs - ex;
        if (qy < 0) qy += g.Ly;
        if (qx < 0) qx += g.Lx;
        const int qi = ch * g.N + qy * g.Lx + qx;
        const double2 zn = cadd(Z2[qi], dzs[q]);
        Z2[qi] = zn;
        RL[qi] = clogcosh(zn).x;
      }
      for (int e = tid; e < g.C * kk; e += 256) {
        const int ch = e / kk, tp = e % kk, dy = tp / g.k, dx = tp % g.k;
        const int p = shift_pos(g, site, -dy, -dx);
        a1[ch * g.N + p] = cadd(a1[ch * g.N + p], DA[e]);
      }
      __syncthreads();
      if (tid == 0) cb[site >> 6] ^= 1ull << (site & 63);
    }
    __syncthreads();
    if (step >= therm_steps && ((step - therm_steps + 1) % sweep) == 0) {
      const int64_t kr = (step - therm_steps + 1) / sweep - 1;
      const int64_t row = kr * n_chains + c;
      for (int w = tid; w < g.W; w += 256) s_out[row * g.W + w] = cb[w];
      double2 lp = make_double2(0.0, 0.0);
      for (int e = tid; e < CN; e += 256) lp = cadd(lp, clogcosh(Z2[e]));
      lp = block_sum(lp, red);
      if (tid == 0 && logpsi_out) logpsi_out[row] = lp;
    }
  }
  for (int w = tid; w < g.W; w += 256) bits[(int64_t)c * g.W + w] = cb[w];
  if (tid == 0) acc[c] = accepted;
}

constexpr int MH_NT = 512, MH_NW = MH_NT / 64;
constexpr int MH_MT = 2;  // column tiles of 16 (tap, output channel) pairs per wave, at most
constexpr int MH_KS = 4;  // k steps of 4 input channels, at most
constexpr int MH_OUT = 2; // window outputs per thread, at most: C (2k-1)^2 <= 784

// Metropolis chains for networks of at most 16 channels and 4 x 4 taps: one
// work-group of eight waves per chain.  A proposal at site f changes z1 at f - t1 and
// z2 at f - t1 - t2; its layer-2 change is one small matrix product
//   P[t1][t2, c] = sum_{c'} dA[t1][c'] W2[c][c'][t2]
// (rows t1, columns (t2, c), no entry wasted at 16 channels and 16 taps) on the float64
// matrix cores, the weights loaded once for the whole launch, followed by the
// window sums dz[c][e] = sum_{t1 + t2 = e} P[t1][t2, c] from LDS.  The acceptance uses
//   Re(log psi' - log psi) = sum (|x'| - |x|) + log(prod q' / prod q) / 2,
//   q = |1 + e^{-2 z~}|^2, z = x + iy, z~ = +-z with real part |x|,
// one logarithm per thread instead of one per output.  State in global memory, channel
// fastest: z1, a1, z2 and q per (position, channel); it is rebuilt from the
// configuration at every launch.  LDS: P (or a1 while the state is built), dA, the
// configuration, and sites and log u of 64 steps drawn at once.
//
// Bound: the latency of four barrier-separated phases per step, with two work-groups on
// a compute unit (their 66 KB of P): the waves wait 48% of their time, the matrix pipe is
// busy 30% of the cycles, vector instructions issue in 38%, and the chains' state moves 22 GB
// through memory, 3.3 TB/s (counters).  The 128 registers of four waves per SIMD do not hold
// everything: 62 of them, with values that a step does not change, lie in scratch memory (140
// bytes a lane) and are read back by up to 18 loads in a step's loop.
// 1 024 chains x 256 steps, 16 x 16, C = 16, k = 4: 84.6 -> 6.52 ms; with four waves a chain,
// whose weights and outputs fit their registers less still, 9.1 ms.
__global__ __launch_bounds__(MH_NT, 4) void k_cnn_mh64(cnn_geom g, int n_chains, int chain0, uint64_t* __restrict__ bits,
                                                     uint2 key, uint64_t t0, int init, int64_t therm_steps,
                                                     int64_t n_record, int sweep, uint64_t* __restrict__ s_out,
                                                     double2* __restrict__ logpsi_out,
                                                     unsigned long long* __restrict__ acc_out,
                                                     double2* __restrict__ scr) {
  extern __shared__ double2 sm[];
  __shared__ double2 DAs[16 * 17];  // dA[t1][c'], rows of 17; zero outside the network
  __shared__ double red[2][MH_NW];
  __shared__ double2 red2[MH_NW];
  __shared__ double lus[64];  // log u
  __shared__ int sites[64];
  __shared__ uint64_t cb[64];
  const int C = g.C, N = g.N, k = g.k, kk = k * k, win = 2 * k - 1, CN = C * N, ld = N + 1;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const int c = chain0 + (int)blockIdx.x;
  const int M = C * kk, MT = (M + 15) / 16, PS = 16 * MT + 1, KS = g.KS;
  double2* P = sm;
  double2* Z1 = scr + (size_t)blockIdx.x * ((7 * (size_t)CN + 1) / 2);
  double2* A1 = Z1 + CN;
  double2* Z2 = A1 + CN;
  double* Q = (double*)(Z2 + CN);
  for (int e = tid; e < 16 * 17; e += MH_NT) DAs[e] = make_double2(0.0, 0.0);
  if (init) {
    if (tid == 0)
      for (int w = 0; w < g.W; ++w) {
        uint4 y = philox(make_uint4((uint32_t)c, (uint32_t)(w >> 1), 0u, 2u), key);
        uint64_t word = (w & 1) ? ((uint64_t)y.z | ((uint64_t)y.w << 32)) : ((uint64_t)y.x | ((uint64_t)y.y << 32));
        const int rem = N - 64 * w;
        if (rem < 64) word &= (1ull << rem) - 1ull;
        cb[w] = word;
      }
  } else {
    for (int w = tid; w < g.W; w += MH_NT) cb[w] = bits[(int64_t)c * g.W + w];
  }
  __syncthreads();
  // the state of the configuration
  const int PT = (N + 15) / 16, PP = (PT + 1) / 2;
  for (int pt = wave; pt < PT; pt += MH_NW) {
    doublex4 re, im;
    z1_tile(g, cb, 0, pt, lane, re, im);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int ch = lk + 4 * r, p = pt * 16 + li;
      if (ch < C && p < N) {
        const double2 z = make_double2(re[r], im[r]), a = clogcosh_pv(z);
        P[ch * ld + p] = a;
        Z1[p * C + ch] = z;
        A1[p * C + ch] = a;
      }
    }
  }
  __syncthreads();
  for (int u = wave; u < PP; u += MH_NW) {
    doublex4 re[2], im[2];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double2 b2 = g.b2[min(lk + 4 * r, C - 1)];
      re[0][r] = re[1][r] = b2.x;
      im[0][r] = im[1][r] = b2.y;
    }
    conv_tiles<2, 1>(g, g.F1, P, ld, 0, 2 * u, lane, re, im);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int ch = lk + 4 * r, p = (2 * u + j) * 16 + li;
        if (ch < C && p < N) {
          const double2 z = make_double2(re[j][r], im[j][r]);
          double2 zt;
          const double2 q = cosh_factor(z, zt);
          Z2[p * C + ch] = z;
          Q[p * C + ch] = fma(q.x, q.x, q.y * q.y);
        }
      }
  }
  // operand columns of this wave's tiles: W2[c][c'][t2] for column (t2, c) = 16 tile + li, c' = 4 ks + lk
  double2 wb[MH_MT][MH_KS];
#pragma unroll
  for (int i = 0; i < MH_MT; ++i)
#pragma unroll
    for (int ks = 0; ks < MH_KS; ++ks) {
      const int m = (wave + MH_NW * i) * 16 + li, t2 = m / C, co = m - t2 * C, ci = 4 * ks + lk;
      wb[i][ks] = (m < M && ci < C) ? g.W2[(co * C + ci) * kk + t2] : make_double2(0.0, 0.0);
    }
  // layer-1 change of this thread: tap t1, channel c1
  const int t1 = tid / C, c1 = tid - t1 * C, dy1 = t1 / k, dx1 = t1 - dy1 * k;
  const bool has1 = tid < M;
  const double2 w1 = has1 ? g.W1[c1 * kk + t1] : make_double2(0.0, 0.0);
  // window outputs of this thread: offsets in the order of their term counts (largest
  // first), so that the lanes of a wave run loops of similar length
  int oe[MH_OUT];  // ey << 16 | ex << 8 | channel
  bool on[MH_OUT]; // outputs past the last repeat it and are left out of the sums
#pragma unroll
  for (int q = 0; q < MH_OUT; ++q) {
    const int o = min(tid + MH_NT * q, C * win * win - 1), r = o / C;
    on[q] = tid + MH_NT * q < C * win * win;
    oe[q] = -1;
    int seen = 0;
    for (int cnt = kk; cnt > 0 && oe[q] < 0; --cnt)
      for (int e = 0; e < win * win; ++e) {
        const int ey = e / win, ex = e - ey * win;
        if (min(ey + 1, win - ey) * min(ex + 1, win - ex) != cnt) continue;
        if (seen++ == r) {
          oe[q] = ey << 16 | ex << 8 | (o - r * C);
          break;
        }
      }
  }
  const double2* p0[MH_OUT];  // first term of the window sum; nx terms PS - C apart, ny rows
  int nyx[MH_OUT];
#pragma unroll
  for (int q = 0; q < MH_OUT; ++q) {
    const int ey = oe[q] >> 16, ex = (oe[q] >> 8) & 255;
    const int ylo = max(0, ey - k + 1), yhi = min(k - 1, ey), xlo = max(0, ex - k + 1), xhi = min(k - 1, ex);
    p0[q] = P + (ylo * k + xlo) * PS + ((ey - ylo) * k + ex - xlo) * C + (oe[q] & 255);
    nyx[q] = (yhi - ylo + 1) << 8 | (xhi - xlo + 1);
  }
  __syncthreads();
  unsigned long long accepted = 0;
  const int64_t total = therm_steps + n_record * sweep;
  for (int64_t step = 0; step < total; ++step) {
    const int sl = (int)(step & 63);
    if (sl == 0) {
      if (tid < 64) {
        const uint64_t t = t0 + (uint64_t)step + (uint64_t)tid;
        const uint4 x = philox(make_uint4((uint32_t)c, (uint32_t)t, (uint32_t)(t >> 32), 0u), key);
        sites[tid] = (int)to_index(x.x, (uint32_t)N);
        lus[tid] = m64::flog(to_uniform(x.y, x.z));
      }
      __syncthreads();
    }
    const int site = __builtin_amdgcn_readfirstlane(sites[sl]);
    const double lu = lus[sl];
    const double ds = -2.0 * sig_at(cb, site);
    int sy, sx;
    pos_yx(g, site, sy, sx);
    // the window's state, in flight over the products
    double2 z2v[MH_OUT];
    double qv[MH_OUT];
    int at[MH_OUT];
#pragma unroll
    for (int q = 0; q < MH_OUT; ++q) {
      int y = sy - (oe[q] >> 16), x = sx - ((oe[q] >> 8) & 255);
      y += y < 0 ? g.Ly : 0;
      x += x < 0 ? g.Lx : 0;
      at[q] = (y * g.Lx + x) * C + (oe[q] & 255);
      z2v[q] = Z2[at[q]];
      qv[q] = Q[at[q]];
    }
    int at1 = 0;
    double2 z1n = make_double2(0.0, 0.0), a1n = z1n;
    if (has1) {
      int y = sy - dy1, x = sx - dx1;
      y += y < 0 ? g.Ly : 0;
      x += x < 0 ? g.Lx : 0;
      at1 = (y * g.Lx + x) * C + c1;
      const double2 z = Z1[at1], a = A1[at1];
      z1n = make_double2(fma(ds, w1.x, z.x), fma(ds, w1.y, z.y));
      a1n = clogcosh_pv(z1n);
      DAs[t1 * 17 + c1] = csub(a1n, a);
    }
    __syncthreads();
    {
      double2 a[MH_KS];
#pragma unroll
      for (int ks = 0; ks < MH_KS; ++ks) a[ks] = DAs[li * 17 + 4 * ks + lk];
#pragma unroll
      for (int i = 0; i < MH_MT; ++i) {
        const int tile = wave + MH_NW * i;
        if (tile >= MT) break;
        doublex4 re0 = doublex4{0.0, 0.0, 0.0, 0.0}, re1 = re0, im0 = re0, im1 = re0;
#pragma unroll
        for (int ks = 0; ks < MH_KS; ++ks) {
          if (ks >= KS) break;
          re0 = mfma64(a[ks].x, wb[i][ks].x, re0);
          im0 = mfma64(a[ks].x, wb[i][ks].y, im0);
          re1 = mfma64(-a[ks].y, wb[i][ks].y, re1);
          im1 = mfma64(a[ks].y, wb[i][ks].x, im1);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (lk + 4 * r < kk)
            P[(lk + 4 * r) * PS + tile * 16 + li] = make_double2(re0[r] + re1[r], im0[r] + im1[r]);
      }
    }
    __syncthreads();
    double2 zn[MH_OUT];
#pragma unroll
    for (int q = 0; q < MH_OUT; ++q) {
      double2 dz = make_double2(0.0, 0.0);
      const double2* row = p0[q];
      for (int y = nyx[q] >> 8; y > 0; --y, row += k * (PS - C)) {
        const double2* pp = row;
        for (int x = nyx[q] & 255; x > 0; --x, pp += PS - C) dz = cadd(dz, *pp);
      }
      zn[q] = cadd(z2v[q], dz);
    }
    double lin = 0.0, num = 1.0, den = 1.0, qn[MH_OUT];
#pragma unroll
    for (int q = 0; q < MH_OUT; ++q) {
      double2 zt;
      const double2 f = cosh_factor(zn[q], zt);
      qn[q] = fma(f.x, f.x, f.y * f.y);
      lin += on[q] ? zt.x - fabs(z2v[q].x) : 0.0;
      num *= on[q] ? qn[q] : 1.0;
      den *= on[q] ? qv[q] : 1.0;
    }
    const double part = wave_sum_uniform(2.0 * lin + m64::flog(m64::fdiv(num, den)));
    if (lane == 0) red[step & 1][wave] = part;
    __syncthreads();
    double r = 0.0;
#pragma unroll
    for (int w = 0; w < MH_NW; ++w) r += red[step & 1][w];
    const bool accept = lu < r;  // r >= 0 or u < e^r
    if (accept) {
      ++accepted;
#pragma unroll
      for (int q = 0; q < MH_OUT; ++q) {
        if (!on[q]) continue;
        Z2[at[q]] = zn[q];
        Q[at[q]] = qn[q];
      }
      if (has1) {
        Z1[at1] = z1n;
        A1[at1] = a1n;
      }
      if (tid == 0) cb[site >> 6] ^= 1ull << (site & 63);
    }
    __syncthreads();
    if (step >= therm_steps && ((step - therm_steps + 1) % sweep) == 0) {
      const int64_t kr = (step - therm_steps + 1) / sweep - 1;
      const int64_t row = kr * n_chains + c;
      for (int w = tid; w < g.W; w += MH_NT) s_out[row * g.W + w] = cb[w];
      if (logpsi_out) {
        double2 lp = make_double2(0.0, 0.0);
        for (int e = tid; e < CN; e += MH_NT) lp = cadd(lp, clogcosh(Z2[e]));
        lp = block_sum(lp, red2);
        if (tid == 0) logpsi_out[row] = lp;
      }
    }
  }
  for (int w = tid; w < g.W; w += MH_NT) bits[(int64_t)c * g.W + w] = cb[w];
  if (tid == 0) acc_out[c] = accepted;
}

constexpr int64_t kChunk = 1 << 14;

cnn_geom geom(const vmc_model* m) {
  cnn_geom g;
  g.Lx = m->Lx;
  g.Ly = m->Ly;
  g.N = m->N;
  g.C = m->C;
  g.k = m->k;
  g.W = m->W;
  const int kk = m->k * m->k;
  g.W1 = m->params;
  g.b1 = m->params + m->C * kk;
  g.W2 = g.b1 + m->C;
  g.b2 = g.W2 + m->C * m->C * kk;
  g.RT = (m->C + 15) / 16;
  g.KS = (m->C + 3) / 4;
  g.KT = (kk + 3) / 4;
  g.F0 = m->cnn_frags;
  g.F1 = g.F0 + (size_t)g.RT * g.KT * 64;
  g.F2 = g.F1 + (size_t)g.RT * kk * g.KS * 64;
  g.invLx = 1.0f / (float)m->Lx;
  return g;
}

size_t lds_limit() { return 160 * 1024; }

template <typename Kern>
void allow_lds(Kern k, size_t bytes) {
  VMC_REQUIRE(bytes <= lds_limit(), "CNN too large for the per-sample LDS budget");
  if (bytes > 64 * 1024) VMC_HIP(hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
}

}  // namespace

size_t cnn_frag_count(const vmc_model* m) {
  const size_t RT = (m->C + 15) / 16, KS = (m->C + 3) / 4, kk = (size_t)m->k * m->k, KT = (kk + 3) / 4;
  return 64 * RT * (KT + 2 * kk * KS);
}

void cnn_set_params(vmc_model* m) {
  const cnn_geom g = geom(m);
  const int64_t n = (int64_t)cnn_frag_count(m), n0 = g.F1 - g.F0, n1 = g.F2 - g.F0;
  k_cnn_frags<<<grid_for(n, 256), 256, 0, m->ctx->stream>>>(g, m->cnn_frags, n0, n1, n);
  VMC_HIP(hipGetLastError());
}

namespace {
// Whether B samples keep the chip busy for more than one round of the work-groups of eight
// waves that the registers leave a compute unit (three of log psi, two of O_k).
bool net_many(const vmc_model* m, int64_t B, bool rows) { return B > (rows ? 2 : 3) * (int64_t)cu_count(m->ctx); }

// Threads of a sample's work-group: two or four waves where layer 2 has as many units (two for
// O_k of one channel up to 256 sites), so that small samples run several groups for each one
// of eight waves, most of which would idle; all eight for few samples, where the latency counts,
// and for larger ones, of which the LDS holds two or three.  8 192 samples, 7 x 7, C = 5, k = 3,
// log psi 258 us with eight waves, 150 with two; O_k of 4 096 samples 5 x 7, C = 5, k = 3 273 and
// 156; 16 x 16, C = 8, k = 1 577 with eight, 798 with two; 64 x 64, C = 1, k = 3, 1 024 samples
// 2.8 and 5.2 ms.
int net_threads(const vmc_model* m, const cnn_geom& g, int64_t B, bool rows) {
  const int u = g.RT * ((g.N + 31) / 32);
  if (!net_many(m, B, rows)) return NET_NT;
  return u <= 2 || (rows && g.C == 1 && u <= 8) ? 128 : u <= 4 ? 256 : NET_NT;
}

size_t net_lds(const cnn_geom& g, int mode) {
  return sizeof(double2) * (size_t)(mode == NET_LOGPSI ? 1 : 2) * g.C * (g.N + 1);
}
}  // namespace

void cnn_log_psi(vmc_model* m, const uint64_t* s, int64_t B, double2* logpsi) {
  const cnn_geom g = geom(m);
  // output by output: one or two channels, which would use a 64th or a 16th of the products (1
  // 024 samples, 16 x 16, k = 4: C = 1 30 against 76 us, C = 2 52 against 77), and few samples
  // of an output a thread whose serial sum is short (16 samples, 5 x 5, C = 9, k = 1 19 against
  // 24 us; 5 x 5, C = 4, k = 4 28 against 24)
  if (g.C <= 2 || (!net_many(m, B, false) && g.C * g.N <= 256 && g.C * g.k * g.k <= 24)) {
    const size_t lds = sizeof(double2) * ((size_t)g.C * g.N + 4);
    allow_lds(k_cnn_forward, lds);
    k_cnn_forward<<<(unsigned)B, 256, lds, m->ctx->stream>>>(g, s, B, logpsi);
    VMC_HIP(hipGetLastError());
    return;
  }
  const size_t lds = net_lds(g, NET_LOGPSI);
  auto run = [&](auto k, int nt) {
    allow_lds(k, lds);
    k<<<(unsigned)B, nt, lds, m->ctx->stream>>>(g, s, B, m->K, nullptr, nullptr, nullptr, logpsi);
    VMC_HIP(hipGetLastError());
  };
  switch (net_threads(m, g, B, false)) {
    case 128: return run(k_cnn_net<NET_LOGPSI, 128, double2>, 128);
    case 256: return run(k_cnn_net<NET_LOGPSI, 256, double2>, 256);
    default: return run(k_cnn_net<NET_LOGPSI, NET_NT, double2>, NET_NT);
  }
}

namespace {
template <typename OutT>
void grad_rows(vmc_model* m, const uint64_t* s, int64_t B, OutT* O) {
  const cnn_geom g = geom(m);
  const size_t lds = net_lds(g, NET_ROWS);
  auto run = [&](auto k, int nt) {
    allow_lds(k, lds);
    k<<<(unsigned)B, nt, lds, m->ctx->stream>>>(g, s, B, m->K, O, nullptr, nullptr, nullptr);
    VMC_HIP(hipGetLastError());
  };
  switch (net_threads(m, g, B, true)) {
    case 128: return run(k_cnn_net<NET_ROWS, 128, OutT>, 128);
    case 256: return run(k_cnn_net<NET_ROWS, 256, OutT>, 256);
    default: return run(k_cnn_net<NET_ROWS, NET_NT, OutT>, NET_NT);
  }
}
}  // namespace

void cnn_grad(vmc_model* m, const uint64_t* s, int64_t B, void* O, int dtype) {
  if (dtype == VMC_DT_C128)
    grad_rows(m, s, B, (double2*)O);
  else
    grad_rows(m, s, B, (float2*)O);
}

void cnn_vjp_partial(vmc_model* m, const uint64_t* s, int64_t B, const double2* gv, int groups, double2* part) {
  const cnn_geom g = geom(m);
  const size_t lds = net_lds(g, NET_VJP);
  auto k = k_cnn_net<NET_VJP, NET_NT, double2>;
  allow_lds(k, lds);
  k<<<(unsigned)groups, NET_NT, lds, m->ctx->stream>>>(g, s, B, m->K, nullptr, gv, part, nullptr);
  VMC_HIP(hipGetLastError());
}

// The (row tile, window offset) units of k_cnn_eloc64 shared out over its waves, the
// costliest first to the least loaded wave: EL_NW + 1 offsets, then rt << 16 | ey << 8 | ex.
// Cost: per pair of taps 4 matrix instructions of 64 cycles and KS steps, per unit about
// 1 600 cycles of vector work.
std::vector<int> cnn_eloc_units(const vmc_model* m) {
  const int k = m->k, win = 2 * k - 1, RT = (m->C + 15) / 16, KS = (m->C + 3) / 4;
  std::vector<std::pair<int, int>> all;
  for (int rt = 0; rt < RT; ++rt)
    for (int ey = 0; ey < win; ++ey)
      for (int ex = 0; ex < win; ++ex) {
        const int pairs = std::min(ey + 1, win - ey) * std::min(ex + 1, win - ex);
        all.push_back({256 * KS * pairs + 1600, rt << 16 | ey << 8 | ex});
      }
  std::stable_sort(all.begin(), all.end(), [](auto& a, auto& b) { return a.first > b.first; });
  std::vector<std::vector<int>> w(EL_NW);
  std::vector<long> load(EL_NW, 0);
  for (auto& u : all) {
    const int q = (int)(std::min_element(load.begin(), load.end()) - load.begin());
    w[q].push_back(u.second);
    load[q] += u.first;
  }
  std::vector<int> out(EL_NW + 1);
  for (int q = 0; q < EL_NW; ++q) {
    out[q] = (int)out.size();
    out.insert(out.end(), w[q].begin(), w[q].end());
  }
  out[EL_NW] = (int)out.size();
  return out;
}

namespace {
constexpr size_t kEl64Fixed = sizeof(double2) * EL_NW * EL_F + sizeof(int) * EL_NW;  // k_cnn_eloc64's own arrays
size_t eloc64_lds(const cnn_geom& g) {
  return sizeof(double2) * (size_t)g.C * ((g.N + 1) + std::max(g.N + 1, g.k * g.k * EL_F));
}

// Local energies through k_cnn_eloc64; false if the sample does not fit its LDS or
// the workspace limit leaves no room for one work-group's scratch.
bool eloc64_run(vmc_model* m, vmc_ham* H, const cnn_geom& g, const uint64_t* s, int64_t B, double2* eloc) {
  vmc_ctx* ctx = m->ctx;
  const size_t lds = eloc64_lds(g);
  if (lds + kEl64Fixed > lds_limit()) return false;
  const int ncu = cu_count(ctx), npass = (g.N + EL_F - 1) / EL_F;
  // one work-group per compute unit; a sample's passes are split over several groups while
  // that fills idle units: rounds of groups x (the forward pass, about one pass, + passes)
  int nsplit = 1;
  double best = INFINITY;
  for (int q = 1; q <= npass; q *= 2) {
    const double t = std::ceil((double)B * q / ncu) * (1.0 + (npass + q - 1) / q);
    if (t < 0.95 * best) {
      best = t;
      nsplit = q;
    }
  }
  const size_t per = ws_round(sizeof(double2) * 3 * (size_t)g.C * g.N);
  const size_t parts = nsplit > 1 ? ws_round(sizeof(double2) * (size_t)B * nsplit) : 0;
  int64_t groups = std::min<int64_t>(B * nsplit, ncu);
  if (ctx->ws_limit) {
    if (ctx->ws_limit < parts + per) return false;
    groups = std::min<int64_t>(groups, (int64_t)((ctx->ws_limit - parts) / per));
  }
  ws_reserve(ctx, per * groups + parts);
  double2* scr = (double2*)ws_take(ctx, per * groups);
  double2* out = nsplit > 1 ? (double2*)ws_take(ctx, sizeof(double2) * (size_t)B * nsplit) : eloc;
  auto launch = [&](auto kern) {
    allow_lds(kern, lds);
    kern<<<(unsigned)groups, EL_NT, lds, ctx->stream>>>(g, s, B, nsplit, H->J, H->h, H->bonds, H->n_bonds,
                                                        m->cnn_units, scr, out);
    VMC_HIP(hipGetLastError());
  };
  if (g.KS == 1)
    launch(k_cnn_eloc64<1>);
  else if (g.KS == 2)
    launch(k_cnn_eloc64<2>);
  else if (g.KS == 3)
    launch(k_cnn_eloc64<3>);
  else if (g.KS == 4)
    launch(k_cnn_eloc64<4>);
  else
    launch(k_cnn_eloc64<0>);
  if (nsplit > 1) {
    k_cnn_eloc_add<<<grid_for(B, 256), 256, 0, ctx->stream>>>(out, B, nsplit, eloc);
    VMC_HIP(hipGetLastError());
  }
  return true;
}
}  // namespace

void cnn_local_energy(vmc_model* m, vmc_ham* H, const uint64_t* s, int64_t B, double2* eloc) {
  VMC_REQUIRE(H->kind == HAM_TFIM, "the CNN local energy supports the transverse-field Ising model");
  VMC_REQUIRE(H->Lx == m->Lx && H->Ly == m->Ly, "lattice of the Hamiltonian differs from the CNN's");
  const cnn_geom g = geom(m);
  const int64_t chunk = std::min<int64_t>(B, kChunk);
  vmc_ctx* ctx = m->ctx;
  if (ctx->ws_limit) ws_reserve(ctx, ws_round(sizeof(double2) * chunk * g.C * g.N));  // the limit of the general kernel
  if (H->h != 0.0 && g.Lx >= 2 * g.k - 1 && g.Ly >= 2 * g.k - 1 && eloc64_run(m, H, g, s, B, eloc)) return;
  const int kk = g.k * g.k;
  const size_t lds = sizeof(double2) * (2 * (size_t)g.C * g.N + (size_t)g.C * kk + 4);
  allow_lds(k_cnn_eloc, lds);
  ws_reserve(ctx, ws_round(sizeof(double2) * chunk * g.C * g.N));
  double2* a1 = (double2*)ws_take(ctx, sizeof(double2) * chunk * g.C * g.N);
  for (int64_t b0 = 0; b0 < B; b0 += chunk) {
    const int64_t nb = std::min(chunk, B - b0);
    k_cnn_eloc<<<(unsigned)nb, 256, lds, ctx->stream>>>(g, s + b0 * g.W, nb, H->J, H->h, H->bonds, H->n_bonds,
                                                        eloc + b0, a1);
    VMC_HIP(hipGetLastError());
  }
}

void cnn_sampler_run(vmc_sampler* S, int64_t n_per_chain, uint64_t* s_out, double2* logpsi_out) {
  vmc_model* m = S->model;
  const cnn_geom g = geom(m);
  VMC_REQUIRE(S->opts.proposal == VMC_PROP_FLIP, "the CNN sampler uses single-spin flips");
  VMC_REQUIRE(g.Lx >= 2 * g.k - 1 && g.Ly >= 2 * g.k - 1, "the CNN sampler needs Lx, Ly >= 2 kernel - 1");
  VMC_REQUIRE(g.C * (2 * g.k - 1) * (2 * g.k - 1) <= 8 * 256, "CNN window too large for the sampler");
  const int CN = g.C * g.N, kk = g.k * g.k;
  vmc_ctx* ctx = S->ctx;
  const int nc = S->opts.n_chains;
  const int64_t therm = S->thermalized ? 0 : (int64_t)S->opts.therm_sweeps * S->opts.sweep_steps;
  const uint2 key = make_uint2((uint32_t)S->opts.seed, (uint32_t)(S->opts.seed >> 32));
  const size_t lds0 = sizeof(double2) * ((size_t)CN + (CN + 1) / 2 + (size_t)g.C * kk + 4) + sizeof(uint64_t) * g.W;
  VMC_REQUIRE(lds0 <= lds_limit(), "CNN too large for the per-sample LDS budget");
  const size_t ws0 = ws_round(sizeof(double2) * (size_t)nc * CN);
  if (ctx->ws_limit) ws_reserve(ctx, ws0);  // the limit of the general kernel
  // Matrix-core chains: up to 16 channels and 4 x 4 taps (one row tile of taps, the weights
  // in the registers of eight waves).  Their state takes 56 bytes per (position, channel), so
  // chains run kMhBatch at a time (32 work-groups a compute unit), or as many as the
  // workspace limit holds; below one, the general kernel, whose scratch is 16 bytes.
  constexpr int64_t kMhBatch = 8192;
  const int MT = (g.C * kk + 15) / 16;
  const size_t lds = sizeof(double2) * std::max<size_t>((size_t)kk * (16 * MT + 1), (size_t)g.C * (g.N + 1));
  const size_t per = sizeof(double2) * ((7 * (size_t)CN + 1) / 2);
  int64_t batch = std::min<int64_t>(nc, kMhBatch);
  if (ctx->ws_limit) batch = std::min<int64_t>(batch, (int64_t)(ctx->ws_limit / per) - 1);
  if (g.C <= 16 && g.k <= 4 && lds + 8192 <= lds_limit() && batch >= 1) {
    allow_lds(k_cnn_mh64, lds);
    ws_reserve(ctx, ws_round(per * batch));
    double2* scr = (double2*)ws_take(ctx, per * batch);
    for (int64_t c0 = 0; c0 < nc; c0 += batch) {
      k_cnn_mh64<<<(unsigned)std::min<int64_t>(batch, nc - c0), MH_NT, lds, ctx->stream>>>(
          g, nc, (int)c0, S->bits, key, S->t, !S->bits_valid, therm, n_per_chain, S->opts.sweep_steps, s_out,
          logpsi_out, S->acc, scr);
      VMC_HIP(hipGetLastError());
    }
  } else {
    allow_lds(k_cnn_metropolis, lds0);
    ws_reserve(ctx, ws0);
    double2* a1 = (double2*)ws_take(ctx, sizeof(double2) * (size_t)nc * CN);
    k_cnn_metropolis<<<nc, 256, lds0, ctx->stream>>>(g, nc, S->bits, key, S->t, !S->bits_valid, therm, n_per_chain,
                                                     S->opts.sweep_steps, s_out, logpsi_out, S->acc, a1);
    VMC_HIP(hipGetLastError());
  }
  S->t += (uint64_t)(therm + n_per_chain * S->opts.sweep_steps);
  S->thermalized = 1;
  S->bits_valid = 1;
}
