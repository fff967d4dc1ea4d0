// RBM network kernels: pre-activations theta = W sigma + b over sample
// batches, log psi, the fused connected-configuration / local-energy kernel,
// and the per-sample log-derivatives O_k.
//
// Local energies (eq:Oloc) need psi(s')/psi(s) on every connected s'.  For the
// RBM of eq:rbm_ex a connected configuration differs from s by one flipped spin
// (TFIM) or one exchanged anti-aligned pair (Heisenberg), i.e. by a "move" m
// that shifts every pre-activation by theta_j -> theta_j - 2 sigma_m D_jm with
//   flip of site l:           D_jm = W_jl,          sigma_m = sigma_l,
//   exchange of bond (i,k):   D_jm = W_ji - W_jk,   sigma_m = sigma_i (= -sigma_k).
// cosh(theta - 2 sigma D) = cosh(theta) cosh(2D) (1 - sigma tanh(theta) tanh(2D)),
// so, exactly,
//   log psi(s') - log psi(s) = -2 sigma_m alpha_m + LC_m + sum_j log(1 - sigma_m t_j T_jm)
// with t_j = tanh(theta_j(s)), T_jm = tanh(2 D_jm), LC_m = sum_j log cosh(2 D_jm)
// and alpha_m = a_l (flip) or a_i - a_k (exchange).  T, LC and alpha depend on
// the parameters only and are tabulated once per parameter version; each
// connected configuration then costs N_h complex multiply-adds and no
// transcendental, instead of a fresh N x N_h network evaluation.
#include "internal.h"

using namespace dev;

namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));

int nh_pad16(int Nh) { return (Nh + 15) / 16 * 16; }
constexpr int kThRows = 64;   // samples per group of the matrix-core theta
constexpr int kThUnits = 32;  // hidden units per group

__device__ __forceinline__ double sign_of(uint64_t w, int i) {  // +1 where bit i is set, else -1
  return __hiloint2double((int)(0xBFF00000u ^ ((uint32_t)(w >> i) << 31)), 0);
}

// theta = b + W sigma on the float64 matrix cores: rows samples, columns units, the
// real and the imaginary part in two accumulators of the same lanes; a group takes 64
// samples x 32 units, a wave 32 x 16.  v_mfma_f64_16x16x4f64: lane l holds
// A[l % 16][l / 16] (sample, site), B[l / 16][l % 16] (site, unit) and, in register r,
// D[l / 16 + 4 r][l % 16].  sigma = +-1 is exact; the sums are float64 in the matrix
// core's order.  Every 16 bytes of W a lane reads feed four products, eight sites'
// reads ahead of them; theta leaves 256 contiguous bytes per 16 lanes.
// Bound: the matrix cores (15 us at 64 sites, 256 units, 16 384 samples) and the write of
// theta (14 us), 36 -> 31 us; 400 sites, 800 units, 4 096 samples 142 -> 122 us (real
// columns of W read 8 bytes at a time, 64 x 64 tiles before).
__global__ __launch_bounds__(256) void k_theta_mfma(const double2* __restrict__ bias, const double2* __restrict__ Wt,
                                                    const uint64_t* __restrict__ s, int64_t B, int N, int W, int Nh,
                                                    double2* __restrict__ theta) {
  extern __shared__ uint64_t sbits[];  // [kThRows][W]
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lk = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t n0 = (int64_t)blockIdx.y * kThRows;
  const int row = 32 * (wv >> 1), unit = blockIdx.x * kThUnits + 16 * (wv & 1) + li;
  for (int e = tid; e < kThRows * W; e += 256) sbits[e] = n0 + e / W < B ? s[n0 * W + e] : 0ull;
  __syncthreads();
  const int ul = unit < Nh ? unit : Nh - 1;  // units past N_h repeat the last, unwritten
  const double2 b = bias[ul];
  doublex4 tr[2], ti[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    tr[h] = doublex4{b.x, b.x, b.x, b.x};
    ti[h] = doublex4{b.y, b.y, b.y, b.y};
  }
  // rows of W of eight steps of four sites; past N: any row (parameters are finite), its
  // product left out
  const double2* col = Wt + ul;
  double2 v[2][8];
  auto load = [&](int k0, double2(&d)[8]) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int i = k0 + 4 * q + lk;
      d[q] = col[(int64_t)(i < N ? i : N - 1) * Nh];
    }
  };
  auto step = [&](int k0, const double2(&d)[8]) {
    const uint64_t w0 = sbits[(row + li) * W + (k0 >> 6)] >> (k0 & 63);
    const uint64_t w1 = sbits[(row + 16 + li) * W + (k0 >> 6)] >> (k0 & 63);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const bool in = k0 + 4 * q + lk < N;
      const double a0 = in ? sign_of(w0, 4 * q + lk) : 0.0, a1 = in ? sign_of(w1, 4 * q + lk) : 0.0;
      tr[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, d[q].x, tr[0], 0, 0, 0);
      ti[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, d[q].y, ti[0], 0, 0, 0);
      tr[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, d[q].x, tr[1], 0, 0, 0);
      ti[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, d[q].y, ti[1], 0, 0, 0);
    }
  };
  load(0, v[0]);
  for (int k0 = 0; k0 < N; k0 += 64) {
    if (k0 + 32 < N) load(k0 + 32, v[1]);
    step(k0, v[0]);
    if (k0 + 32 >= N) break;
    if (k0 + 64 < N) load(k0 + 64, v[0]);
    step(k0 + 32, v[1]);
  }
  if (unit < Nh)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t n = n0 + row + 16 * h + lk + 4 * r;
        if (n < B) theta[n * Nh + unit] = make_double2(tr[h][r], ti[h][r]);
      }
}

// theta of a sample's hidden units as the kernels below take it: from memory
// (k_theta_mfma), or for small calls formed where it is used, which saves the
// launch and the round trip.
struct theta_src {
  const double2* theta;   // [B][N_h], or NULL
  const double2* params;  // for theta == NULL: parameters and transposed weights [N][N_h]
  const double2* Wt;
};

__device__ __forceinline__ double2 theta_at(const theta_src& t, const uint64_t* sn, int64_t n, int N, int Nh, int j) {
  if (t.theta) return t.theta[n * Nh + j];
  double2 th = t.params[N + j];
  for (int i0 = 0; i0 < N; i0 += 64) {
    const uint64_t w = sn[i0 >> 6];
    const double2* col = t.Wt + (int64_t)i0 * Nh + j;
    const int ni = N - i0 < 64 ? N - i0 : 64;
#pragma unroll 8
    for (int i = 0; i < ni; ++i) {
      const double sg = (w >> i) & 1ull ? 1.0 : -1.0;
      const double2 v = col[(int64_t)i * Nh];
      th = make_double2(fma(sg, v.x, th.x), fma(sg, v.y, th.y));
    }
  }
  return th;
}

// log psi of many samples with theta in registers only: 32 samples per work-group, wave w
// the unit tiles w, w + 4, ... of 16 units.  theta = b + sigma W is a product on the
// float64 matrix cores (rows samples, columns units, real and imaginary parts in two
// accumulators of the same lanes), so that a lane takes log cosh of its own entries and
// adds them up over its tiles; the weights of the next 64 sites or tile are on their way
// while it does.
// Bound: the matrix cores and the elementary functions, one after the other.  N = 64,
// N_h = 256, 16 384 samples 71 -> 58 us (theta through memory before).
__global__ __launch_bounds__(256, 2) void k_logpsi_mfma(const double2* __restrict__ params,
                                                        const double2* __restrict__ Wt,
                                                        const uint64_t* __restrict__ s, int64_t B, int N, int W,
                                                        int Nh, double2* __restrict__ logpsi) {
  extern __shared__ uint64_t bits[];  // [32][W]
  __shared__ double2 ths[4][4][64];  // theta of four of a lane's eight entries
  __shared__ double2 lps[4][8][64];  // and their sums of log cosh over the tiles
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lk = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t n0 = (int64_t)blockIdx.x * 32;
  for (int e = tid; e < 32 * W; e += 256) bits[e] = n0 + e / W < B ? s[n0 * W + e] : 0ull;
  __syncthreads();
  // entry (site, unit) of the weights; sites past N read zero, units past N_h the next site's
  // (their log cosh is left out).  The hardware takes a lane's offset as out of range from
  // (range - scalar offset) on: the scalar one may not pass the range itself
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)Wt, 0, N * Nh * 16, 0x00027000);
  double2 v[16];
  auto load = [&](int ut, int w) {
    const int at = (lk * Nh + ut * 16 + li) * 16;
#pragma unroll
    for (int q = 0; q < 16; ++q)
      v[q] = __builtin_bit_cast(double2,
                                __builtin_amdgcn_raw_buffer_load_b128(rsrc, at, min(64 * w + 4 * q, N) * Nh * 16, 0));
  };
  const int ntile = (Nh + 15) / 16;
#pragma unroll
  for (int e = 0; e < 8; ++e) lps[wv][e][lane] = make_double2(0.0, 0.0);
  if (wv < ntile) load(wv, 0);
  for (int ut = wv; ut < ntile; ut += 4) {
    const int unit = ut * 16 + li;
    double2 b = make_double2(0.0, 0.0);
    if (unit < Nh) b = params[N + unit];
    doublex4 tr[2], ti[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      tr[h] = doublex4{b.x, b.x, b.x, b.x};
      ti[h] = doublex4{b.y, b.y, b.y, b.y};
    }
    for (int w = 0; w < W; ++w) {
      const uint64_t w0 = bits[li * W + w], w1 = bits[(16 + li) * W + w];
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const double a0 = sign_of(w0, 4 * q + lk), a1 = sign_of(w1, 4 * q + lk);
        tr[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, v[q].x, tr[0], 0, 0, 0);
        ti[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, v[q].y, ti[0], 0, 0, 0);
        tr[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, v[q].x, tr[1], 0, 0, 0);
        ti[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, v[q].y, ti[1], 0, 0, 0);
      }
      if (w + 1 < W)
        load(ut, w + 1);
      else if (ut + 4 < ntile)
        load(ut + 4, 0);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int r = 0; r < 4; ++r) ths[wv][r][lane] = make_double2(tr[h][r], ti[h][r]);
      if (unit < Nh)
#pragma unroll 1
        for (int r = 0; r < 4; ++r)
          lps[wv][4 * h + r][lane] = cadd(lps[wv][4 * h + r][lane], clogcosh(ths[wv][r][lane]));
    }
  }
  // sum_i a_i sigma_i, eight threads per sample
  double2 va = make_double2(0.0, 0.0);
  for (int i = tid & 7; i < N; i += 8) {
    const uint64_t w = bits[(tid >> 3) * W + (i >> 6)];
    va = cadd(va, cscale(params[i], sign_of(w, i & 63)));
  }
#pragma unroll
  for (int o = 1; o < 8; o <<= 1) {
    va.x += __shfl_xor(va.x, o, 64);
    va.y += __shfl_xor(va.y, o, 64);
  }
  // sample 16 h + 4 r + k: entry 4 h + r of lanes 16 k .. 16 k + 15 of the four waves, two
  // lanes of each wave per thread
  __syncthreads();
  const int q = tid >> 3, part = tid & 7;
  double2 l = make_double2(0.0, 0.0);
#pragma unroll
  for (int w = 0; w < 4; ++w)
#pragma unroll
    for (int u = 0; u < 2; ++u)
      l = cadd(l, lps[w][4 * (q >> 4) + ((q & 15) >> 2)][16 * (q & 3) + 2 * part + u]);
#pragma unroll
  for (int o = 1; o < 8; o <<= 1) {
    l.x += __shfl_xor(l.x, o, 64);
    l.y += __shfl_xor(l.y, o, 64);
  }
  if (part == 0 && n0 + q < B) logpsi[n0 + q] = cadd(va, l);
}

// log psi(n) = sum_i a_i sigma_i + sum_j logcosh(theta_j); one wave per sample.
__global__ __launch_bounds__(64) void k_logpsi(const double2* __restrict__ params, theta_src theta,
                                               const uint64_t* __restrict__ s, int64_t B, int N, int W, int Nh,
                                               double2* __restrict__ logpsi) {
  const int64_t n = blockIdx.x;
  if (n >= B) return;
  const int lane = threadIdx.x;
  double2 acc = make_double2(0.0, 0.0);
  const uint64_t* sn = s + n * W;
  for (int i = lane; i < N; i += 64) {
    const double2 a = params[i];
    const double sg = get_bit(sn, i) ? 1.0 : -1.0;
    acc = cadd(acc, cscale(a, sg));
  }
  for (int j = lane; j < Nh; j += 64) acc = cadd(acc, clogcosh(theta_at(theta, sn, n, N, Nh, j)));
  acc = wave_sum(acc);
  if (lane == 0) logpsi[n] = acc;
}

// Move tables: one wave per move m.
// T and D [N_h][n_moves]; T holds zero rows past N_h up to Nhp (a multiple of 16)
__global__ __launch_bounds__(64) void k_tables(const double2* __restrict__ params, const int2* __restrict__ bonds,
                                               int move_kind, int n_moves, int N, int Nh, int Nhp, double2* __restrict__ T,
                                               double2* __restrict__ D, double2* __restrict__ LC,
                                               double2* __restrict__ alpha) {
  const int m = blockIdx.x;
  if (m >= n_moves) return;
  const int lane = threadIdx.x;
  const double2* Wm = params + N + Nh;
  int i, k = -1;
  if (move_kind == 0) {
    i = m;
  } else {
    i = bonds[m].x;
    k = bonds[m].y;
  }
  double2 lc = make_double2(0.0, 0.0);
  for (int j = lane; j < Nh; j += 64) {
    double2 d = Wm[(int64_t)j * N + i];
    if (k >= 0) d = csub(d, Wm[(int64_t)j * N + k]);
    const double2 d2 = cscale(d, 2.0);
    D[(int64_t)j * n_moves + m] = d;
    T[(int64_t)j * n_moves + m] = ctanh(d2);
    lc = cadd(lc, clogcosh(d2));
  }
  for (int j = Nh + lane; j < Nhp; j += 64) T[(int64_t)j * n_moves + m] = make_double2(0.0, 0.0);
  lc = wave_sum(lc);
  if (lane == 0) {
    LC[m] = lc;
    alpha[m] = k >= 0 ? csub(params[i], params[k]) : params[i];
  }
}

// Entry (unit, move) of the move table T [Nhp][n_moves] (at most 2^23 entries): the unit's row
// as scalar offset, the move as lane offset, so that a row costs no vector arithmetic
__device__ __forceinline__ __amdgpu_buffer_rsrc_t table_rsrc(const double2* T, int Nhp, int n_moves) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)T, 0, Nhp * n_moves * 16, 0x00027000);
}
__device__ __forceinline__ double2 table_at(__amdgpu_buffer_rsrc_t rsrc, int unit, int n_moves, int m) {
  return __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(rsrc, m * 16, unit * n_moves * 16, 0));
}

// Local energies, S samples per wavefront, for move sets shared by all samples
// (single-spin flips of the TFIM; the kernel also accepts bonds, masked per
// sample to the anti-aligned ones).  Lanes run over the moves, and every table
// entry T_jm read from memory serves the S samples, whose tanh theta_j sit in
// LDS.  For each (sample,
// move) the product prod_j (1 - sigma t_j T_jm) is kept with exact
// power-of-two rescaling, and
//   E_loc = diag + mel * sum_m exp(-2 sigma_m alpha_m + LC_m + log prod).
// Bound: float64 vector work, ten instructions per (unit, move).  The padded table and
// operands need no bounds, and its rows are addressed from scalar registers, U of them in
// flight: N = 64, N_h = 256, 16 384 samples with theta 237 -> 200 us.
template <int S, int U>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(U == 16 ? 2 : 1, U == 16 ? 2 : 8))) void k_eloc(theta_src theta, const uint64_t* __restrict__ s,
                                             int64_t B, int N, int W, int Nh, int ham_kind, double J, double h,
                                             const int2* __restrict__ bonds, int n_bonds,
                                             const double2* __restrict__ T, const double2* __restrict__ LC,
                                             const double2* __restrict__ alpha, int n_moves, int Nhp,
                                             double2* __restrict__ eloc) {
  extern __shared__ double2 tl[];  // [S][Nhp], 0 past N_h
  const int64_t b0 = (int64_t)blockIdx.x * S;
  if (b0 >= B) return;
  const int lane = threadIdx.x;
#pragma unroll
  for (int q = 0; q < S; ++q)
    for (int j = lane; j < Nhp; j += 64)
      tl[q * Nhp + j] = b0 + q < B && j < Nh ? ctanh(theta_at(theta, s + (b0 + q) * W, b0 + q, N, Nh, j)) : make_double2(0.0, 0.0);
  // diagonal element: coupling * (n_aligned - n_anti), exact integer count
  double diag[S];
#pragma unroll
  for (int q = 0; q < S; ++q) {
    int n_al = 0;
    if (b0 + q < B) {
      const uint64_t* sn = s + (b0 + q) * W;
      for (int b = lane; b < n_bonds; b += 64) {
        const int2 bd = bonds[b];
        n_al += get_bit(sn, bd.x) == get_bit(sn, bd.y);
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) n_al += __shfl_xor(n_al, o, 64);
    const int n_anti = n_bonds - n_al;
    diag[q] = ham_kind == HAM_TFIM ? -J * (double)(n_al - n_anti) : J * (double)(n_al - n_anti);
  }
  __syncthreads();
  const auto rsrc = table_rsrc(T, Nhp, n_moves);
  const double mel = ham_kind == HAM_TFIM ? -h : 2.0 * J;
  const bool off = ham_kind == HAM_TFIM ? h != 0.0 : J != 0.0;
  double2 acc[S];
#pragma unroll
  for (int q = 0; q < S; ++q) acc[q] = make_double2(0.0, 0.0);
  if (off)
    for (int m0 = 0; m0 < n_moves; m0 += 64) {
      const int m = m0 + lane;
      if (m >= n_moves) continue;
      const int site = ham_kind == HAM_TFIM ? m : bonds[m].x;
      const int site2 = ham_kind == HAM_TFIM ? -1 : bonds[m].y;
      double sg[S];
      bool active[S];
      double2 P[S];
      int e2[S];
#pragma unroll
      for (int q = 0; q < S; ++q) {
        const bool in = b0 + q < B;
        const uint64_t* sn = s + (in ? b0 + q : b0) * W;
        const int bi = get_bit(sn, site);
        sg[q] = bi ? 1.0 : -1.0;
        active[q] = in && (site2 < 0 || bi != get_bit(sn, site2));
        P[q] = make_double2(1.0, 0.0);
        e2[q] = 0;
      }
      for (int j0 = 0; j0 < Nhp; j0 += 16) {  // T and tl are 0 past N_h
#pragma unroll
        for (int jb = j0; jb < j0 + 16; jb += U) {
          double2 Tv[U];  // U rows in flight before the products that use them
#pragma unroll
          for (int u = 0; u < U; ++u) Tv[u] = table_at(rsrc, jb + u, n_moves, m);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int u = 0; u < U; ++u)
#pragma unroll
            for (int q = 0; q < S; ++q) {
              const double2 tt = cmul(tl[q * Nhp + jb + u], Tv[u]);
              P[q] = cmul(P[q], make_double2(fma(-sg[q], tt.x, 1.0), -sg[q] * tt.y));
            }
        }
        // keep |P| within 2^-64 .. 2^64 (from there sixteen factors of 1e-18 to 1e18 stay in
        // range): exact power-of-two rescaling of the wave's products once one has left it
        bool far = false;
#pragma unroll
        for (int q = 0; q < S; ++q)
          far |= (uint32_t)__double2hiint(fmax(fabs(P[q].x), fabs(P[q].y))) - ((1023u - 64u) << 20) > 128u << 20;
        if (__ballot(far))
#pragma unroll
          for (int q = 0; q < S; ++q) {
            const int e = __builtin_amdgcn_frexp_exp(fmax(fabs(P[q].x), fabs(P[q].y)));
            P[q] = make_double2(ldexp(P[q].x, -e), ldexp(P[q].y, -e));
            e2[q] += e;
          }
      }
      const double2 al = alpha[m], lcm = LC[m];
#pragma unroll
      for (int q = 0; q < S; ++q) {
        if (!active[q]) continue;
        double2 lr = cadd(cscale(al, -2.0 * sg[q]), lcm);
        // log |P| = log of the mantissa + exponent log 2
        const int e = __builtin_amdgcn_frexp_exp(fmax(fabs(P[q].x), fabs(P[q].y)));
        const double2 lp = clog(make_double2(ldexp(P[q].x, -e), ldexp(P[q].y, -e)));
        lr.x += lp.x + (double)(e2[q] + e) * 0.69314718055994530942;
        lr.y += lp.y;
        acc[q] = cadd(acc[q], cscale(cexp(lr), mel));
      }
    }
#pragma unroll
  for (int q = 0; q < S; ++q) {
    const double2 v = wave_sum(acc[q]);
    if (lane == 0 && b0 + q < B) eloc[b0 + q] = make_double2(v.x + diag[q], v.y);
  }
}

// Fused enumeration + evaluation + reduction of E_loc, one wave per sample, for
// move sets that depend on the sample (exchanges of anti-aligned bonds).
// Bound: the table reads' latency and float64 vector work.  U rows and operands are in
// flight before their products; 4 096 samples, ring of 64 sites: 256 units 75 us with eight,
// 78 with sixteen, 600 units 161 and 141, 1 024 units 318 and 287 (reads interleaved by the
// compiler, about eight in flight: 78, 178 and 379).
// LDS: t_j (Nh complex) and the compacted move list (<= n_moves ints).
template <int U>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(U == 16 ? 2 : 1, U == 16 ? 2 : 8))) void k_eloc_compact(theta_src theta, const uint64_t* __restrict__ s,
                                             int64_t B, int N, int W, int Nh, int ham_kind, double J, double h,
                                             const int2* __restrict__ bonds, int n_bonds,
                                             const double2* __restrict__ T, const double2* __restrict__ LC,
                                             const double2* __restrict__ alpha, int n_moves, int Nhp,
                                             double2* __restrict__ eloc) {
  // sigma t_j for both spins: tpm[0][j] = -t_j, tpm[1][j] = t_j, zero past N_h up
  // to Nhp (a multiple of 16, where the table rows are zero as well)
  extern __shared__ double2 lds[];
  double2* tpm = lds;                            // [2][Nhp]
  int* moves = (int*)(lds + 2 * Nhp);            // [n_moves]
  const int64_t n = blockIdx.x;
  if (n >= B) return;
  const int lane = threadIdx.x;
  const uint64_t* sn = s + n * W;

  for (int j = lane; j < Nhp; j += 64) {
    const double2 tj = j < Nh ? ctanh(theta_at(theta, sn, n, N, Nh, j)) : make_double2(0.0, 0.0);
    tpm[j] = make_double2(-tj.x, -tj.y);
    tpm[Nhp + j] = tj;
  }

  const auto rsrc = table_rsrc(T, Nhp, n_moves);
  // diagonal element: coupling * (n_aligned - n_anti), exact integer count
  int n_al = 0;
  for (int b = lane; b < n_bonds; b += 64) {
    const int2 bd = bonds[b];
    n_al += get_bit(sn, bd.x) == get_bit(sn, bd.y);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) n_al += __shfl_xor(n_al, o, 64);
  const int n_anti = n_bonds - n_al;
  const double diag = ham_kind == HAM_TFIM ? -J * (double)(n_al - n_anti) : J * (double)(n_al - n_anti);

  // compacted list of off-diagonal moves in slot order
  int n_slots = 0;
  double mel;
  if (ham_kind == HAM_TFIM) {
    mel = -h;
    if (h != 0.0) {
      for (int l = lane; l < N; l += 64) moves[l] = l;
      n_slots = N;
    }
  } else {
    mel = 2.0 * J;
    if (J != 0.0) {
      for (int b0 = 0; b0 < n_bonds; b0 += 64) {
        const int b = b0 + lane;
        bool anti = false;
        if (b < n_bonds) {
          const int2 bd = bonds[b];
          anti = get_bit(sn, bd.x) != get_bit(sn, bd.y);
        }
        const uint64_t mask = __ballot(anti);
        const int pos = n_slots + __popcll(mask & ((1ull << lane) - 1ull));
        if (anti) moves[pos] = b;
        n_slots += __popcll(mask);
      }
    }
  }
  __syncthreads();

  double2 acc = make_double2(0.0, 0.0);
  for (int q0 = 0; q0 < n_slots; q0 += 64) {
    const int q = q0 + lane;
    if (q < n_slots) {
      const int m = moves[q];
      const int site = ham_kind == HAM_TFIM ? m : bonds[m].x;
      const int up = get_bit(sn, site);
      const double sg = up ? 1.0 : -1.0;
      const double2* st = tpm + (up ? Nhp : 0);  // sigma t of this slot's spin
      double2 P = make_double2(1.0, 0.0);
      int e2 = 0;
      for (int j0 = 0; j0 < Nhp; j0 += 16) {
#pragma unroll
        for (int jb = j0; jb < j0 + 16; jb += U) {
          double2 Tv[U], tv[U];  // U rows and operands in flight before their products
#pragma unroll
          for (int u = 0; u < U; ++u) Tv[u] = table_at(rsrc, jb + u, n_moves, m);
#pragma unroll
          for (int u = 0; u < U; ++u) tv[u] = st[jb + u];
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const double2 tt = cmul(tv[u], Tv[u]);  // sigma t_j T_jm
            P = cmul(P, make_double2(1.0 - tt.x, -tt.y));
          }
        }
        // keep |P| near 1: exact power-of-two rescaling
        int e;
        frexp(fmax(fabs(P.x), fabs(P.y)), &e);
        P.x = ldexp(P.x, -e);
        P.y = ldexp(P.y, -e);
        e2 += e;
      }
      const double2 a = alpha[m];
      double2 lr = cadd(cscale(a, -2.0 * sg), LC[m]);
      const double2 lp = clog(P);
      lr.x += lp.x + (double)e2 * 0.69314718055994530942;
      lr.y += lp.y;
      acc = cadd(acc, cscale(cexp(lr), mel));
    }
  }
  acc = wave_sum(acc);
  if (lane == 0) eloc[n] = make_double2(acc.x + diag, acc.y);
}

// O_k rows: [sigma (N), t (Nh), t_j sigma_i (Nh x N)]; one block per sample.
template <typename OutT>
__global__ __launch_bounds__(256) void k_grad(theta_src theta, const uint64_t* __restrict__ s,
                                              int64_t B, int N, int W, int Nh, int64_t K, OutT* __restrict__ O) {
  extern __shared__ double2 tl[];  // [Nh]
  const int64_t n = blockIdx.x;
  if (n >= B) return;
  const int tid = threadIdx.x;
  const uint64_t* sn = s + n * W;
  for (int j = tid; j < Nh; j += 256) tl[j] = ctanh(theta_at(theta, sn, n, N, Nh, j));
  __syncthreads();
  OutT* row = O + n * K;
  auto put = [&](int64_t k, double2 v) {
    if constexpr (sizeof(OutT) == sizeof(double2))
      row[k] = v;
    else
      row[k] = make_float2((float)v.x, (float)v.y);
  };
  for (int i = tid; i < N; i += 256) put(i, make_double2(get_bit(sn, i) ? 1.0 : -1.0, 0.0));
  for (int j = tid; j < Nh; j += 256) put(N + j, tl[j]);
  const int64_t nw = (int64_t)N * Nh;
  for (int64_t e = tid; e < nw; e += 256) {
    const int j = (int)(e / N);
    const int i = (int)(e - (int64_t)j * N);
    const double2 v = tl[j];
    put(N + Nh + e, get_bit(sn, i) ? v : make_double2(-v.x, -v.y));
  }
}

// get_s_primes as a test export: one thread per sample.
__global__ void k_connected(const uint64_t* __restrict__ s, int64_t B, int N, int W, int ham_kind, double J,
                            double h, const int2* __restrict__ bonds, int n_bonds, int M_max,
                            uint64_t* __restrict__ sp, double* __restrict__ mel, int32_t* __restrict__ count) {
  const int64_t n = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (n >= B) return;
  const uint64_t* sn = s + n * W;
  int n_al = 0;
  for (int b = 0; b < n_bonds; ++b) n_al += get_bit(sn, bonds[b].x) == get_bit(sn, bonds[b].y);
  const int n_anti = n_bonds - n_al;
  uint64_t* out = sp + n * (int64_t)M_max * W;
  double* me = mel + n * (int64_t)M_max;
  auto copy_s = [&](int slot) {
    for (int w = 0; w < W; ++w) out[(int64_t)slot * W + w] = sn[w];
  };
  copy_s(0);
  me[0] = ham_kind == HAM_TFIM ? -J * (double)(n_al - n_anti) : J * (double)(n_al - n_anti);
  int c = 1;
  if (ham_kind == HAM_TFIM) {
    if (h != 0.0)
      for (int l = 0; l < N; ++l, ++c) {
        copy_s(c);
        out[(int64_t)c * W + (l >> 6)] ^= 1ull << (l & 63);
        me[c] = -h;
      }
  } else if (J != 0.0) {
    for (int b = 0; b < n_bonds; ++b) {
      const int i = bonds[b].x, k = bonds[b].y;
      if (get_bit(sn, i) == get_bit(sn, k)) continue;
      copy_s(c);
      out[(int64_t)c * W + (i >> 6)] ^= 1ull << (i & 63);
      out[(int64_t)c * W + (k >> 6)] ^= 1ull << (k & 63);
      me[c] = 2.0 * J;
      ++c;
    }
  }
  count[n] = c;
  for (int q = c; q < M_max; ++q) {
    copy_s(q);
    me[q] = 0.0;
  }
}

constexpr int64_t kChunk = 1 << 16;  // samples per theta chunk

}  // namespace

void rbm_theta(vmc_model* m, const uint64_t* s, int64_t B, double2* theta, hipStream_t st) {
  if (!st) st = m->ctx->stream;
  // at most 65535 row tiles per launch
  const int64_t chunk = (int64_t)65535 * kThRows;
  const unsigned gx = (unsigned)((m->Nh + kThUnits - 1) / kThUnits);
  for (int64_t b0 = 0; b0 < B; b0 += chunk) {
    const int64_t nb = std::min(chunk, B - b0);
    k_theta_mfma<<<dim3(gx, (unsigned)((nb + kThRows - 1) / kThRows)), 256, sizeof(uint64_t) * kThRows * m->W, st>>>(
        m->params + m->N, m->Wt, s + b0 * m->W, nb, m->N, m->W, m->Nh, theta + b0 * m->Nh);
    VMC_HIP(hipGetLastError());
  }
}

namespace {
// where the kernels take theta of B samples at s from: `buf`, filled here, or for
// small calls their own loop.  That loop reads N rows of W per 64 units in batches of
// eight and B N N_h entries in all, against a launch and theta's round trip (3 to 5 us):
// the line is where either would cost about as much (64 rows; 2^22 entries, 64 MB from
// the caches; 8 192 samples).  Log psi, local energies and O_k, 1 024 samples: N = N_h =
// 10 31.9 -> 20.9 us, N = N_h = 64 60.5 -> 39.6 us, N = 30, N_h = 120 53.3 -> 42.7 us;
// 16 384 samples of N = N_h = 6 would gain 2 us in each of the first two and lose 3 in
// the last.
theta_src take_theta(vmc_model* m, const uint64_t* s, int64_t B, double2* buf) {
  if ((int64_t)m->N * ((m->Nh + 63) / 64) <= 64 && B <= 8192 && B * m->N * m->Nh <= (int64_t)1 << 22)
    return {nullptr, m->params, m->Wt};
  rbm_theta(m, s, B, buf);
  return {buf, nullptr, nullptr};
}

// [rows][cols] -> [cols][rows] for two tables at once (sampler layout)
__global__ void k_transpose2(const double2* __restrict__ A, const double2* __restrict__ B, int rows, int cols,
                             double2* __restrict__ At, double2* __restrict__ Bt) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= (int64_t)rows * cols) return;
  const int64_t r = e / cols, c = e % cols;
  At[c * rows + r] = A[e];
  Bt[c * rows + r] = B[e];
}
}  // namespace

void rbm_ensure_tables(vmc_model* m, const vmc_ham* H, int move_kind) {
  rbm_move_tables& tb = m->tab[move_kind];
  const int n_moves = move_kind == 0 ? m->N : H->n_bonds;
  if (tb.T && tb.param_version == m->version && tb.n_moves == n_moves && (move_kind == 0 || tb.ham_uid == H->uid)) return;
  if (tb.n_moves != n_moves || !tb.T) {
    VMC_HIP(hipStreamSynchronize(m->ctx->stream));
    if (tb.T) VMC_HIP(hipFree(tb.T));
    if (tb.D) VMC_HIP(hipFree(tb.D));
    if (tb.LC) VMC_HIP(hipFree(tb.LC));
    if (tb.alpha) VMC_HIP(hipFree(tb.alpha));
    if (tb.Tt) VMC_HIP(hipFree(tb.Tt));
    if (tb.Dt) VMC_HIP(hipFree(tb.Dt));
    tb.T = tb.D = tb.LC = tb.alpha = tb.Tt = tb.Dt = nullptr;
    size_t tsz = sizeof(double2) * (size_t)m->Nh * std::max(1, n_moves);
    VMC_HIP(hipMalloc(&tb.T, sizeof(double2) * (size_t)nh_pad16(m->Nh) * std::max(1, n_moves)));
    VMC_HIP(hipMalloc(&tb.D, tsz));
    VMC_HIP(hipMalloc(&tb.Tt, tsz));
    VMC_HIP(hipMalloc(&tb.Dt, tsz));
    VMC_HIP(hipMalloc(&tb.LC, sizeof(double2) * std::max(1, n_moves)));
    VMC_HIP(hipMalloc(&tb.alpha, sizeof(double2) * std::max(1, n_moves)));
  }
  tb.move_kind = move_kind;
  tb.n_moves = n_moves;
  tb.ham_uid = H->uid;
  if (n_moves > 0) {
    k_tables<<<n_moves, 64, 0, m->ctx->stream>>>(m->params, H->bonds, move_kind, n_moves, m->N, m->Nh,
                                                 nh_pad16(m->Nh), tb.T, tb.D, tb.LC, tb.alpha);
    const int64_t n = (int64_t)m->Nh * n_moves;
    k_transpose2<<<grid_for(n, 256), 256, 0, m->ctx->stream>>>(tb.T, tb.D, m->Nh, n_moves, tb.Tt, tb.Dt);
    VMC_HIP(hipGetLastError());
  }
  tb.param_version = m->version;
}

// log psi from theta of the same configurations
void rbm_log_psi_theta(vmc_model* m, const uint64_t* s, int64_t B, const double2* theta, double2* logpsi) {
  k_logpsi<<<(unsigned)B, 64, 0, m->ctx->stream>>>(m->params, theta_src{theta, nullptr, nullptr}, s, B, m->N, m->W,
                                                  m->Nh, logpsi);
  VMC_HIP(hipGetLastError());
}

void rbm_log_psi(vmc_model* m, const uint64_t* s, int64_t B, double2* logpsi) {
  vmc_ctx* ctx = m->ctx;
  const int64_t chunk = std::min<int64_t>(B, kChunk);
  ws_reserve(ctx, ws_round(sizeof(double2) * chunk * m->Nh));
  double2* theta = (double2*)ws_take(ctx, sizeof(double2) * chunk * m->Nh);
  for (int64_t b0 = 0; b0 < B; b0 += chunk) {
    const int64_t nb = std::min(chunk, B - b0);
    // in registers where 32 samples per group give every compute unit one (N = 64, N_h =
    // 256: 8 192 samples 40 against 53 us) and the weights' offsets fit 31 bits (the spins of up
    // to 4 096 sites fit the LDS beside 48 KB of sums)
    if (nb >= 32 * (int64_t)cu_count(ctx) && (int64_t)(m->N + 64) * m->Nh * 16 < (int64_t)1 << 31) {
      k_logpsi_mfma<<<(unsigned)((nb + 31) / 32), 256, sizeof(uint64_t) * 32 * m->W, ctx->stream>>>(
          m->params, m->Wt, s + b0 * m->W, nb, m->N, m->W, m->Nh, logpsi + b0);
      VMC_HIP(hipGetLastError());
      continue;
    }
    const theta_src th = take_theta(m, s + b0 * m->W, nb, theta);
    k_logpsi<<<(unsigned)nb, 64, 0, ctx->stream>>>(m->params, th, s + b0 * m->W, nb, m->N, m->W, m->Nh, logpsi + b0);
    VMC_HIP(hipGetLastError());
  }
}

void rbm_local_energy(vmc_model* m, vmc_ham* H, const uint64_t* s, int64_t B, double2* eloc) {
  vmc_ctx* ctx = m->ctx;
  const int move_kind = H->kind == HAM_TFIM ? 0 : 1;
  rbm_ensure_tables(m, H, move_kind);
  const rbm_move_tables& tb = m->tab[move_kind];
  const int64_t chunk = std::min<int64_t>(B, kChunk);
  ws_reserve(ctx, ws_round(sizeof(double2) * chunk * m->Nh));
  double2* theta = (double2*)ws_take(ctx, sizeof(double2) * chunk * m->Nh);
  // flips: 4 samples per wavefront share the table reads where that leaves two waves per
  // SIMD (B >= 8 192) of which four fit the LDS (N_h <= 256) and fill their lanes (more
  // than 32 moves): N = 64, N_h = 256: 204 against 220 us for 16 384 samples with one
  // each; otherwise one sample: N = 400, N_h = 800, 4 096 samples 1.08 against 2.15 ms,
  // N = 10, N_h = 10, 1 024 samples 12 against 20 us.  Exchanges: one sample per wavefront
  // over its compacted list of anti-aligned bonds.
  const int S = nh_pad16(m->Nh) <= 256 && tb.n_moves > 32 && B >= 8192 ? 4 : 1;
  const int Nhp = nh_pad16(m->Nh);
  const size_t lds = sizeof(double2) * (size_t)S * Nhp;
  const size_t lds1 = sizeof(double2) * 2 * Nhp + sizeof(int) * std::max(1, tb.n_moves);
  VMC_REQUIRE((move_kind == 1 ? lds1 : lds) <= 64 * 1024, "model too large for the local-energy kernel's LDS budget");
  VMC_REQUIRE((int64_t)Nhp * std::max(1, tb.n_moves) < ((int64_t)1 << 31), "move table too large");
  for (int64_t b0 = 0; b0 < B; b0 += chunk) {
    const int64_t nb = std::min(chunk, B - b0);
    const theta_src th = take_theta(m, s + b0 * m->W, nb, theta);
    if (move_kind == 1) {
      // rows of T in flight: eight, and sixteen above 256 units, where the LDS rather than the
      // registers limits the waves and the reads' latency shows
#define COMPACT_LAUNCH(UU)                                                                                          \
  k_eloc_compact<UU><<<(unsigned)nb, 64, lds1, ctx->stream>>>(th, s + b0 * m->W, nb, m->N, m->W, m->Nh, H->kind,    \
                                                              H->J, H->h, H->bonds, H->n_bonds, tb.T, tb.LC,        \
                                                              tb.alpha, tb.n_moves, Nhp, eloc + b0)
      if (Nhp <= 256)
        COMPACT_LAUNCH(8);
      else
        COMPACT_LAUNCH(16);
#undef COMPACT_LAUNCH
      VMC_HIP(hipGetLastError());
      continue;
    }
    const unsigned grid = (unsigned)((nb + S - 1) / S);
    // rows of T in flight: eight, and sixteen above 512 units, where the LDS leaves a SIMD two
    // or three waves (400 sites, 800 units, 4 096 samples 990 against 1 066 us; 100 sites, 400
    // units 176 against 170)
#define ELOC_LAUNCH(SS, UU)                                                                                        \
  k_eloc<SS, UU><<<grid, 64, lds, ctx->stream>>>(th, s + b0 * m->W, nb, m->N, m->W, m->Nh, H->kind, H->J, H->h,    \
                                                 H->bonds, H->n_bonds, tb.T, tb.LC, tb.alpha, tb.n_moves, Nhp,     \
                                                 eloc + b0)
    if (S == 4)
      ELOC_LAUNCH(4, 8);
    else if (Nhp <= 512)
      ELOC_LAUNCH(1, 8);
    else
      ELOC_LAUNCH(1, 16);
#undef ELOC_LAUNCH
    VMC_HIP(hipGetLastError());
  }
}

void rbm_grad(vmc_model* m, const uint64_t* s, int64_t B, void* O, int dtype) {
  vmc_ctx* ctx = m->ctx;
  const int64_t chunk = std::min<int64_t>(B, kChunk);
  ws_reserve(ctx, ws_round(sizeof(double2) * chunk * m->Nh));
  double2* theta = (double2*)ws_take(ctx, sizeof(double2) * chunk * m->Nh);
  const size_t esz = dtype == VMC_DT_C128 ? sizeof(double2) : sizeof(float2);
  for (int64_t b0 = 0; b0 < B; b0 += chunk) {
    const int64_t nb = std::min(chunk, B - b0);
    const theta_src th = take_theta(m, s + b0 * m->W, nb, theta);
    void* out = (char*)O + (size_t)b0 * m->K * esz;
    if (dtype == VMC_DT_C128)
      k_grad<double2><<<(unsigned)nb, 256, sizeof(double2) * m->Nh, ctx->stream>>>(
          th, s + b0 * m->W, nb, m->N, m->W, m->Nh, m->K, (double2*)out);
    else
      k_grad<float2><<<(unsigned)nb, 256, sizeof(double2) * m->Nh, ctx->stream>>>(
          th, s + b0 * m->W, nb, m->N, m->W, m->Nh, m->K, (float2*)out);
    VMC_HIP(hipGetLastError());
  }
}

void ham_connected_impl(vmc_ham* H, const uint64_t* s, int64_t B, uint64_t* sp, double* mel, int32_t* cnt) {
  k_connected<<<grid_for(B, 128), 128, 0, H->ctx->stream>>>(s, B, H->N, H->W, H->kind, H->J, H->h, H->bonds,
                                                             H->n_bonds, H->M_max, sp, mel, cnt);
  VMC_HIP(hipGetLastError());
}
