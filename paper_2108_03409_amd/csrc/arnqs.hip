// Autoregressive neural quantum state with direct sampling (Sec. 2.4: the joint
// distribution factorises into conditionals p_i(s_i | s_<i), so a sample is drawn
// site by site with one network pass and no Markov chain).
//
// The state is psi(s) = sqrt(q(s)) with q a masked autoregressive network (MADE:
// one ReLU hidden layer, hidden degree m(k) = k mod (N - 1) + 1, W1 entry (k, d)
// live iff m(k) >= d + 1, W2 entry (i, k) live iff i + 1 > m(k)), so log psi =
// (1/2) sum_i [s_i l_i - softplus(l_i)] is real and psi is normalised over all 2^N
// configurations.  The parameter vector holds only the live entries, in the order
//   W1 (k ascending, then d < m(k)) | b1 (H) | W2 (i ascending, then k with m(k) <= i) | b2 (N),
// N H + H + N real numbers; masked weights are not parameters.
//
// Local energies (eq:Oloc) use the move structure of the network: flipping or
// swapping sites P changes the hidden pre-activations by the W1 columns of P, and
// only the logits i >= min P can change, so each connected configuration costs one
// sparse hidden update and one (N - min P) x H product instead of a full pass.
// O_k = d log psi / d theta_k is the per-sample backward pass of the same network.
#include <hip/hip_runtime.h>

#include <type_traits>
#include <vector>

#include "internal.h"

using namespace dev;

namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));

constexpr int AR_NT = 256;
constexpr int AR_WAVES = AR_NT / 64;

__device__ __forceinline__ int ar_deg(int k, int N) { return k % (N - 1) + 1; }
__device__ __forceinline__ double ar_softplus(double x) { return fmax(x, 0.0) + log1p(exp(-fabs(x))); }

// value of `v` in lane `src` (src uniform across the wave); reads the register
// whatever the execution mask, so every lane must have written it
__device__ __forceinline__ double lane_bcast(double v, int src) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, src);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), src);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// One configuration through the network, all threads of the group:
// x (N, 0/1), a (H, pre-activations), hh (H, ReLU), l (N, logits).
__device__ void ar_forward(const uint64_t* __restrict__ srow, int N, int H, const double* __restrict__ W1mT,
                           const double* __restrict__ W2t, const double* __restrict__ b1,
                           const double* __restrict__ b2, double* x, double* a, double* hh, double* l) {
  for (int d = threadIdx.x; d < N; d += AR_NT) x[d] = (double)((srow[d >> 6] >> (d & 63)) & 1ull);
  __syncthreads();
  for (int k = threadIdx.x; k < H; k += AR_NT) {
    double acc = b1[k];
    const int m = ar_deg(k, N);
    for (int d = 0; d < m; ++d) acc = fma(W1mT[(int64_t)d * H + k], x[d], acc);
    a[k] = acc;
    hh[k] = fmax(acc, 0.0);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < N; i += AR_NT) {
    double acc = b2[i];
    for (int k = 0; k < H; ++k) acc = fma(W2t[(int64_t)k * N + i], hh[k], acc);
    l[i] = acc;
  }
  __syncthreads();
}

__global__ __launch_bounds__(AR_NT) void k_ar_log_psi(const uint64_t* __restrict__ s, int N, int H, int W,
                                                      const double* __restrict__ W1mT, const double* __restrict__ W2t,
                                                      const double* __restrict__ b1, const double* __restrict__ b2,
                                                      double2* __restrict__ out) {
  extern __shared__ double lds[];
  __shared__ double red[AR_WAVES];
  double *x = lds, *a = x + N, *hh = a + H, *l = hh + H;
  const int64_t b = blockIdx.x;
  ar_forward(s + b * W, N, H, W1mT, W2t, b1, b2, x, a, hh, l);
  double acc = 0.0;
  // where a bit agrees with its logit the first bracket is exactly 0 and the sum keeps
  // the relative precision of its small terms
  for (int i = threadIdx.x; i < N; i += AR_NT)
    acc += (x[i] * l[i] - fmax(l[i], 0.0)) - log1p(exp(-fabs(l[i])));
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < AR_WAVES; ++w) t += red[w];
    out[b] = make_double2(0.5 * t, 0.0);
  }
}

// E_loc of one configuration per group.  Wave 0 lists the connected moves in the
// canonical slot order (TFIM: every site when h != 0; Heisenberg: anti-aligned
// bonds in bond order when J != 0) and counts aligned bonds for the diagonal; the
// four waves then take moves round-robin, lanes over hidden units for the update
// of the pre-activations and over outputs i >= min P for the new logits.
template <int QH>
__global__ __launch_bounds__(AR_NT) void k_ar_eloc(const uint64_t* __restrict__ s, int N, int H, int W,
                                                   const double* __restrict__ W1mT, const double* __restrict__ W2t,
                                                   const double* __restrict__ b1, const double* __restrict__ b2,
                                                   int kind, double J, double hx, const int2* __restrict__ bonds,
                                                   int n_bonds, double2* __restrict__ eloc) {
  extern __shared__ double lds[];
  __shared__ double red[AR_WAVES];
  __shared__ int n_moves_s, n_al_s;
  double *x = lds, *a = x + N, *hh = a + H, *l = hh + H, *t = l + N;
  int* mv = (int*)(t + N);
  const int64_t b = blockIdx.x;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  ar_forward(s + b * W, N, H, W1mT, W2t, b1, b2, x, a, hh, l);
  for (int i = threadIdx.x; i < N; i += AR_NT) t[i] = x[i] * l[i] - ar_softplus(l[i]);
  if (wave == 0) {
    const uint64_t* srow = s + b * W;
    int n_al = 0, nm = 0;
    const bool list = kind == HAM_HEIS && J != 0.0;
    for (int b0 = 0; b0 < n_bonds; b0 += 64) {
      const int q = b0 + lane;
      bool al = false, anti = false;
      if (q < n_bonds) {
        const int2 bd = bonds[q];
        al = get_bit(srow, bd.x) == get_bit(srow, bd.y);
        anti = !al;
      }
      n_al += __popcll(__ballot(al));
      const unsigned long long am = __ballot(anti);
      if (list && anti) mv[nm + __popcll(am & ((1ull << lane) - 1ull))] = q;
      nm += __popcll(am);
    }
    if (lane == 0) {
      n_al_s = n_al;
      n_moves_s = kind == HAM_TFIM ? (hx != 0.0 ? N : 0) : (list ? nm : 0);
    }
  }
  __syncthreads();
  const int M = n_moves_s;
  const double mel = kind == HAM_TFIM ? -hx : 2.0 * J;
  double e_w = 0.0;
  for (int mi = wave; mi < M; mi += AR_WAVES) {
    int p0, p1;
    if (kind == HAM_TFIM) {
      p0 = mi;
      p1 = -1;
    } else {
      const int2 bd = bonds[mv[mi]];
      p0 = min(bd.x, bd.y);
      p1 = max(bd.x, bd.y);
    }
    const double d0 = 1.0 - 2.0 * x[p0];
    const double d1 = p1 >= 0 ? 1.0 - 2.0 * x[p1] : 0.0;
    double dh[QH];
#pragma unroll
    for (int q = 0; q < QH; ++q) {
      const int k = lane + 64 * q;
      dh[q] = 0.0;
      if (k < H) {
        double ap = fma(W1mT[(int64_t)p0 * H + k], d0, a[k]);
        if (p1 >= 0) ap = fma(W1mT[(int64_t)p1 * H + k], d1, ap);
        dh[q] = fmax(ap, 0.0) - hh[k];
      }
    }
    double acc = 0.0;
    for (int i0 = p0; i0 < N; i0 += 64) {  // uniform trip count
      const int i = i0 + lane;
      const bool ok = i < N;
      double lp = ok ? l[i] : 0.0;
#pragma unroll
      for (int q = 0; q < QH; ++q) {
        for (int kk = 0; kk < 64; ++kk) {
          const int k = 64 * q + kk;
          if (k >= H) break;
          const double d = lane_bcast(dh[q], kk);
          if (d != 0.0 && ok) lp = fma(W2t[(int64_t)k * N + i], d, lp);
        }
      }
      if (ok) {
        const double xi = (i == p0 || i == p1) ? 1.0 - x[i] : x[i];
        acc += (xi * lp - ar_softplus(lp)) - t[i];
      }
    }
    acc = wave_sum(acc);
    e_w += mel * exp(0.5 * acc);
  }
  if (lane == 0) red[wave] = e_w;
  __syncthreads();
  if (threadIdx.x == 0) {
    const int n_anti = n_bonds - n_al_s;
    const double diag = (kind == HAM_TFIM ? -J : J) * (double)(n_al_s - n_anti);
    double e = diag;
    for (int w = 0; w < AR_WAVES; ++w) e += red[w];
    eloc[b] = make_double2(e, 0.0);
  }
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// O_k = (1/2) d log q / d theta_k for SB configurations per group:
//   g_l[i] = s_i - sigmoid(l_i),  g_h[k] = [a_k > 0] sum_i (W2 * M2)[i, k] g_l[i],
//   W1 (k, d): g_h[k] s_d,  b1 k: g_h[k],  W2 (i, k): g_l[i] relu(a_k),  b2 i: g_l[i].
template <int SB, typename OutT>
__global__ __launch_bounds__(AR_NT) void k_ar_grad(const uint64_t* __restrict__ s, int64_t B, int N, int H, int W,
                                                   const double* __restrict__ W1mT, const double* __restrict__ W2t,
                                                   const double* __restrict__ W2m, const double* __restrict__ b1,
                                                   const double* __restrict__ b2, const int2* __restrict__ idx,
                                                   int64_t r1, int64_t r2, int64_t r3, int64_t K,
                                                   OutT* __restrict__ O) {
  extern __shared__ double lds[];
  const int per = 2 * N + 3 * H;
  const int64_t b0 = (int64_t)blockIdx.x * SB;
  for (int q = 0; q < SB; ++q) {
    double* x = lds + q * per;
    double *a = x + N, *hh = a + H, *l = hh + H, *gh = l + N;
    if (b0 + q < B) {  // uniform over the group
      ar_forward(s + (b0 + q) * W, N, H, W1mT, W2t, b1, b2, x, a, hh, l);
      for (int i = threadIdx.x; i < N; i += AR_NT) l[i] = x[i] - 1.0 / (1.0 + exp(-l[i]));
      __syncthreads();
      for (int k = threadIdx.x; k < H; k += AR_NT) {
        double acc = 0.0;
        for (int i = ar_deg(k, N); i < N; ++i) acc = fma(W2m[(int64_t)i * H + k], l[i], acc);
        gh[k] = a[k] > 0.0 ? acc : 0.0;
      }
      __syncthreads();
    }
  }
  for (int64_t j = threadIdx.x; j < K; j += AR_NT) {
    const int2 pr = idx[j];
    const int region = j < r1 ? 0 : j < r2 ? 1 : j < r3 ? 2 : 3;
#pragma unroll
    for (int q = 0; q < SB; ++q) {
      if (b0 + q >= B) break;
      const double* x = lds + q * per;
      const double *a = x + N, *hh = a + H, *gl = hh + H, *gh = gl + N;
      (void)a;
      double v;
      if (region == 0)
        v = gh[pr.x] * x[pr.y];
      else if (region == 1)
        v = gh[pr.x];
      else if (region == 2)
        v = gl[pr.x] * hh[pr.y];
      else
        v = gl[pr.x];
      v *= 0.5;
      OutT* row = O + (b0 + q) * K;
      if constexpr (std::is_same<OutT, double2>::value)
        row[j] = make_double2(v, 0.0);
      else if constexpr (std::is_same<OutT, float2>::value)
        row[j] = make_float2((float)v, 0.0f);
      else
        row[j] = (OutT)v;
    }
  }
}

// O_k with the weights in LDS and a configuration per wave, for networks that fit 64 KB: a
// wave writes whole rows and needs no other wave.  Bound: the serial sums of its hidden units.
template <typename OutT>
__global__ __launch_bounds__(AR_NT) void k_ar_grad_w(const uint64_t* __restrict__ s, int64_t B, int N, int H, int W,
                                                     const double* __restrict__ W1mT,
                                                     const double* __restrict__ W2t, const double* __restrict__ b1,
                                                     const double* __restrict__ b2, const int2* __restrict__ idx,
                                                     int64_t r1, int64_t r2, int64_t r3, int64_t K,
                                                     OutT* __restrict__ O) {
  extern __shared__ double lds[];
  double* W1s = lds;          // [N][H]
  double* W2s = W1s + N * H;  // [H][N]
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  double* x = W2s + H * N + wave * (2 * N + 2 * H);
  double* gl = x + N;   // logits, then s_i - sigmoid(l_i)
  double* hh = gl + N;  // ReLU(a), with a kept as the sign of the gate below
  double* gh = hh + H;
  for (int e = threadIdx.x; e < N * H; e += AR_NT) {
    W1s[e] = W1mT[e];
    W2s[e] = W2t[e];
  }
  __syncthreads();
  for (int64_t b = (int64_t)blockIdx.x * AR_WAVES + wave; b < B; b += (int64_t)gridDim.x * AR_WAVES) {
    const uint64_t* srow = s + b * W;
    for (int i = lane; i < N; i += 64) x[i] = (double)((srow[i >> 6] >> (i & 63)) & 1ull);
    wave_sync();
    for (int k = lane; k < H; k += 64) {
      double acc = b1[k];
      for (int d = 0; d < N; ++d) acc = fma(W1s[d * H + k], x[d], acc);
      hh[k] = fmax(acc, 0.0);
      gh[k] = acc > 0.0 ? 1.0 : 0.0;  // ReLU gate
    }
    wave_sync();
    for (int i = lane; i < N; i += 64) {
      double acc = b2[i];
      for (int k = 0; k < H; ++k) acc = fma(W2s[k * N + i], hh[k], acc);
      gl[i] = x[i] - 1.0 / (1.0 + exp(-acc));
    }
    wave_sync();
    for (int k = lane; k < H; k += 64) {
      double acc = 0.0;
      for (int i = ar_deg(k, N); i < N; ++i) acc = fma(W2s[k * N + i], gl[i], acc);
      gh[k] *= acc;
    }
    wave_sync();
    OutT* row = O + b * K;
    for (int64_t j = lane; j < K; j += 64) {
      const int2 pr = idx[j];
      double v;
      if (j < r1)
        v = gh[pr.x] * x[pr.y];
      else if (j < r2)
        v = gh[pr.x];
      else if (j < r3)
        v = gl[pr.x] * hh[pr.y];
      else
        v = gl[pr.x];
      v *= 0.5;
      if constexpr (std::is_same<OutT, double2>::value)
        row[j] = make_double2(v, 0.0);
      else if constexpr (std::is_same<OutT, float2>::value)
        row[j] = make_float2((float)v, 0.0f);
      else
        row[j] = (OutT)v;
    }
    wave_sync();
  }
}

// ---- 16 configurations per work-group on the float64 matrix cores -----------
// The network of a batch of 16 configurations is three small products on 16 x 16 x 4
// operands (lane l holds A[l % 16][l / 16], B[l / 16][l % 16] and, in register r,
// D[l / 16 + 4 r][l % 16]):
//   a[n][k] = b1 + sum_d x[n][d] W1[d][k],   l[n][i] = b2 + sum_k relu(a) W2[k][i],
//   g_h[n][k] = sum_i g_l[n][i] W2[k][i].
// Hidden units are stored by ascending degree, so the units that a flip of site p
// changes (degree > p) and the units that output i reads (degree <= i) are ranges of
// positions, and the reduction of a block runs over their intersection only.
// Weights in LDS, zero past the network; the row lengths keep 16 rows apart in the
// banks.
struct ar_net {
  int N, H, W;
  int NT1, NT2;      // tiles of 16 hidden units / outputs
  int Hs, Ns;        // row lengths of W1 [4 ceil(N / 4)][Hs] and W2 [16 NT1][Ns]
  int pm;            // sites p < pm change some hidden unit
  const double* pad; // W1 | W2 | b1 [Hs] | b2 [Ns]
  const int* mst;    // [N + 1]: first position of degree >= v
  __host__ __device__ int n4() const { return (N + 3) / 4 * 4; }
  __host__ __device__ int w_doubles() const { return n4() * Hs + 16 * NT1 * Ns + Hs + Ns; }
};

constexpr int AB = 16;  // configurations per batch
constexpr int AB_NT = 512, AB_WAVES = AB_NT / 64;

struct ar_lds {
  double *W1, *W2, *b1, *b2;
  int* mst;       // [N + 1]
  double *a;      // [AB][Hs] pre-activations
  double *l;      // [AB][Ns] logits (or g_l)
  double *x2;     // [AB][Ns] 1 + e^{-|l|} (local energies) or [AB][Hs] g_h (gradients)
  uint64_t* bits; // [AB][W]
};

__host__ __device__ inline size_t ar_lds_doubles(const ar_net& d, int x2) {
  return d.w_doubles() + (size_t)AB * (d.Hs + d.Ns + x2 + d.W) + (d.N + 2) / 2;
}

__device__ __forceinline__ ar_lds ar_lds_at(const ar_net& d, double* p, int x2) {
  ar_lds L;
  L.W1 = p;
  L.W2 = L.W1 + d.n4() * d.Hs;
  L.b1 = L.W2 + 16 * d.NT1 * d.Ns;
  L.b2 = L.b1 + d.Hs;
  L.mst = (int*)(L.b2 + d.Ns);
  L.a = L.b2 + d.Ns + (d.N + 2) / 2;
  L.l = L.a + AB * d.Hs;
  L.x2 = L.l + AB * d.Ns;
  L.bits = (uint64_t*)(L.x2 + AB * x2);
  return L;
}

__device__ __forceinline__ void ar_load(const ar_net& d, const ar_lds& L) {
  const int n = d.w_doubles();
  for (int e = threadIdx.x; e < n; e += AB_NT) L.W1[e] = d.pad[e];
  for (int e = threadIdx.x; e <= d.N; e += AB_NT) L.mst[e] = d.mst[e];
}

__device__ __forceinline__ doublex4 mfma64(double a, double b, doublex4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ double ar_bit(const ar_net& d, const ar_lds& L, int n, int i) {
  return (double)((L.bits[n * d.W + (i >> 6)] >> (i & 63)) & 1ull);
}

// Bits and pre-activations of configurations b0 .. b0 + 15 (repeating the last past B)
// into LDS, by the group (ends with a barrier) or, WAVE, by one wave with a batch of its own.
template <bool WAVE>
__device__ __forceinline__ void ar_hidden16(const ar_net& d, const ar_lds& L, const uint64_t* __restrict__ s,
                                            int64_t b0, int64_t B) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
  for (int e = WAVE ? lane : threadIdx.x; e < AB * d.W; e += WAVE ? 64 : AB_NT) {
    const int n = e / d.W;
    L.bits[e] = s[min(b0 + n, B - 1) * d.W + e - n * d.W];
  }
  if (WAVE)
    wave_sync();
  else
    __syncthreads();
  const uint64_t* row = L.bits + li * d.W;
  for (int nt = WAVE ? 0 : wave; nt < d.NT1; nt += WAVE ? 1 : AB_WAVES) {
    const double b = L.b1[16 * nt + li];
    doublex4 acc = doublex4{b, b, b, b};
    for (int k0 = 0; k0 < d.N; k0 += 4) {
      const int i = k0 + lk;  // rows of W1 past N are 0
      const double x = i < d.N ? (double)((row[i >> 6] >> (i & 63)) & 1ull) : 0.0;
      acc = mfma64(x, L.W1[i * d.Hs + 16 * nt + li], acc);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) L.a[(lk + 4 * r) * d.Hs + 16 * nt + li] = acc[r];
  }
  if (WAVE)
    wave_sync();
  else
    __syncthreads();
}

// Logits of the batch at outputs 16 nt + li: register r is configuration lk + 4 r.
__device__ __forceinline__ doublex4 ar_logits16(const ar_net& d, const ar_lds& L, int nt, int li, int lk) {
  const double b = L.b2[16 * nt + li];
  doublex4 acc = doublex4{b, b, b, b};
  const int ke = L.mst[min(d.N, 16 * nt + 16)];  // units of degree <= 16 nt + 15
  for (int k0 = 0; k0 < ke; k0 += 4) {
    const int k = k0 + lk;
    acc = mfma64(fmax(L.a[li * d.Hs + k], 0.0), L.W2[k * d.Ns + 16 * nt + li], acc);
  }
  return acc;
}

// log psi, a batch per wave: the softplus sum as one logarithm of prod (1 + e^{-|l|}) per
// configuration (the product of N <= 512 factors in [1, 2] stays in range), held as its
// excess over 1, p <- p + x + p x, so that saturated conditionals (x far below 2^-53) keep
// their relative precision.  Bound: the latency of the products and of one exponential per
// logit.  3e5 configurations, N = 50, H = 29: 0.81 -> 0.10 ms (0.21 ms with a batch per group).
__global__ __launch_bounds__(AB_NT, 4) void k_ar_log_psi16(ar_net d, const uint64_t* __restrict__ s, int64_t B,
                                                           double2* __restrict__ out) {
  extern __shared__ double lds[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
  ar_lds L = ar_lds_at(d, lds, 0);
  ar_load(d, L);
  __syncthreads();
  L.bits = (uint64_t*)(lds + d.w_doubles() + (d.N + 2) / 2) + wave * AB * (d.W + d.Hs);  // after weights and mst
  L.a = (double*)(L.bits + AB * d.W);
  const int64_t step = (int64_t)gridDim.x * AB_WAVES * AB;
  for (int64_t b0 = ((int64_t)blockIdx.x * AB_WAVES + wave) * AB; b0 < B; b0 += step) {
    ar_hidden16<true>(d, L, s, b0, B);
    double lin[4] = {0.0, 0.0, 0.0, 0.0}, q[4] = {0.0, 0.0, 0.0, 0.0};
    for (int nt = 0; nt < d.NT2; ++nt) {
      const doublex4 l = ar_logits16(d, L, nt, li, lk);
      const int i = 16 * nt + li;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double x = ar_bit(d, L, lk + 4 * r, min(i, d.N - 1));
        lin[r] += i < d.N ? x * l[r] - fmax(l[r], 0.0) : 0.0;
        const double e = m64::fexp_neg0(l[r]);
        q[r] = i < d.N ? q[r] + fma(q[r], e, e) : q[r];
      }
    }
    double a = 0.0, p = 0.0;  // lane li < 4: configuration lk + 4 li
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double ar = row16_sum(lin[r]), pr = row16_excess(q[r]);
      if (li == r) {
        a = ar;
        p = pr;
      }
    }
    if (li < 4 && b0 + lk + 4 * li < B) out[b0 + lk + 4 * li] = make_double2(0.5 * (a - m64::flog1p(p)), 0.0);
    wave_sync();  // the batch's LDS is rewritten by the next one
  }
}

// Local energies.  The forward pass as above; then a wave takes a configuration's connected
// moves 16 at a time: the changes of the hidden units (rows: moves) times W2 give the new
// logits as one product with the old logits as its start, over the units of degree > the
// smallest site of the block, for the outputs from that site on.  Per entry one exponential:
//   2 (log psi' - log psi) = sum_i [x' l' - max(l', 0) - x l + max(l, 0)] - log(prod q' / prod q),
//   q = 1 + e^{-|l|}, with one logarithm per move.  Flips that change no unit (TFIM, p >= pm)
// need no product and no q.
// Bound: float64 vector work (the exponentials).  3e5 configurations, N = 50, H = 29, TFIM:
// 7.09 -> 1.81 ms (one wave per configuration with (move, output) pairs over its lanes, both
// weight operands of every multiply-add from LDS, exp and log1p per pair).
__global__ __launch_bounds__(AB_NT, 4) void k_ar_eloc16(ar_net d, const uint64_t* __restrict__ s, int64_t B, int kind,
                                                     double J, double hx, const int2* __restrict__ bonds, int n_bonds,
                                                     double2* __restrict__ eloc) {
  extern __shared__ double lds[];
  const ar_lds L = ar_lds_at(d, lds, d.Ns);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  int* mv = (int*)(L.bits + AB * d.W) + wave * n_bonds;  // anti-aligned bonds (Heisenberg), bond order
  const double mel = kind == HAM_TFIM ? -hx : 2.0 * J;
  const bool offdiag = kind == HAM_TFIM ? hx != 0.0 : J != 0.0;
  ar_load(d, L);
  for (int64_t b0 = (int64_t)blockIdx.x * AB; b0 < B; b0 += (int64_t)gridDim.x * AB) {
    __syncthreads();
    ar_hidden16<false>(d, L, s, b0, B);
    for (int nt = wave; nt < d.NT2; nt += AB_WAVES) {
      const doublex4 l = ar_logits16(d, L, nt, li, lk);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        L.l[(lk + 4 * r) * d.Ns + 16 * nt + li] = l[r];
        L.x2[(lk + 4 * r) * d.Ns + 16 * nt + li] = 1.0 + m64::fexp_neg0(l[r]);
      }
    }
    __syncthreads();
    for (int n = wave; n < AB && b0 + n < B; n += AB_WAVES) {
      const uint64_t* brow = L.bits + n * d.W;
      const double *an = L.a + n * d.Hs, *ln = L.l + n * d.Ns, *qn = L.x2 + n * d.Ns;
      int n_al = 0, M = 0;
      for (int q0 = 0; q0 < n_bonds; q0 += 64) {
        const int q = q0 + lane;
        bool al = false, anti = false;
        if (q < n_bonds) {
          const int2 bd = bonds[q];
          al = get_bit(brow, bd.x) == get_bit(brow, bd.y);
          anti = !al;
        }
        n_al += __popcll(__ballot(al));
        const unsigned long long am = __ballot(anti);
        if (kind == HAM_HEIS && anti) mv[M + __popcll(am & ((1ull << lane) - 1ull))] = q;
        M += __popcll(am);
      }
      if (kind == HAM_TFIM) M = d.pm;
      if (!offdiag) M = 0;
      wave_sync();
      double e = 0.0;
      if (offdiag && kind == HAM_TFIM)
        for (int p = d.pm + lane; p < d.N; p += 64) e += m64::fexp(0.5 * (1.0 - 2.0 * get_bit(brow, p)) * ln[p]);
      for (int m0 = 0; m0 < M; m0 += 16) {
        // this lane's row of the block: move m0 + li
        int p0 = d.N, p1 = -1;
        if (m0 + li < M) {
          p0 = m0 + li;
          if (kind == HAM_HEIS) {
            const int2 bd = bonds[mv[m0 + li]];
            p0 = min(bd.x, bd.y);
            p1 = max(bd.x, bd.y);
          }
        }
        const bool ok = p0 < d.N;
        const int pc0 = min(p0, d.N - 1), pc1 = max(p1, 0);
        const double d0 = ok ? 1.0 - 2.0 * get_bit(brow, pc0) : 0.0, d1 = p1 >= 0 ? 1.0 - 2.0 * get_bit(brow, pc1) : 0.0;
        int pmin = m0;
        if (kind == HAM_HEIS) {
          pmin = p0;
          for (int o = 8; o > 0; o >>= 1) pmin = min(pmin, __shfl_xor(pmin, o, 64));
          pmin = __builtin_amdgcn_readfirstlane(pmin);
        }
        int r0[4], r1[4];  // sites of the lane's accumulator rows
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          r0[r] = __shfl(p0, lk + 4 * r, 64);
          r1[r] = kind == HAM_HEIS ? __shfl(p1, lk + 4 * r, 64) : -1;
        }
        double lin[4] = {0.0, 0.0, 0.0, 0.0}, num[4] = {1.0, 1.0, 1.0, 1.0}, den[4] = {1.0, 1.0, 1.0, 1.0};
        const int ks = __builtin_amdgcn_readfirstlane(L.mst[pmin + 1]) & ~3;
        for (int n0 = pmin >> 4; n0 < d.NT2; n0 += 4) {
          const int ne = min(4, d.NT2 - n0);
          const int ke = __builtin_amdgcn_readfirstlane(L.mst[min(d.N, 16 * (n0 + ne))]);
          doublex4 acc[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const double l = j < ne ? ln[16 * (n0 + j) + li] : 0.0;
            acc[j] = doublex4{l, l, l, l};
          }
          for (int k0 = ks; k0 < ke; k0 += 4) {
            const int k = k0 + lk;
            const double av = an[k];
            double ap = fma(L.W1[pc0 * d.Hs + k], d0, av);
            if (kind == HAM_HEIS) ap = fma(L.W1[pc1 * d.Hs + k], d1, ap);
            const double dh = fmax(ap, 0.0) - fmax(av, 0.0);  // 0 for units of degree <= p0
            const double* w2 = L.W2 + k * d.Ns + 16 * n0 + li;
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if (j < ne) acc[j] = mfma64(dh, w2[16 * j], acc[j]);
          }
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            if (j >= ne) break;
            const int i = 16 * (n0 + j) + li, ic = min(i, d.N - 1);
            const double x = (double)get_bit(brow, ic), l = ln[i], q = qn[i];
            const double t = x * l - fmax(l, 0.0);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const bool in = i >= r0[r] && i < d.N;
              const double lp = acc[j][r], xp = (i == r0[r] || i == r1[r]) ? 1.0 - x : x;
              lin[r] += in ? (xp * lp - fmax(lp, 0.0)) - t : 0.0;
              if (ke > ks) {
                num[r] *= in ? 1.0 + m64::fexp_neg0(lp) : 1.0;
                den[r] *= in ? q : 1.0;
              }
            }
          }
        }
        double la = 0.0, ra = 1.0;  // lane li < 4: the sums of row lk + 4 li
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const double a = row16_sum(lin[r]), p = row16_prod(m64::fdiv(num[r], den[r]));
          if (li == r) {
            la = a;
            ra = p;
          }
        }
        if (li < 4 && m0 + lk + 4 * li < M) e += m64::fexp(0.5 * (la - m64::flog(ra)));
      }
      e = wave_sum_uniform(e);
      if (lane == 0) {
        const int n_anti = n_bonds - n_al;
        const double diag = (kind == HAM_TFIM ? -J : J) * (double)(n_al - n_anti);
        eloc[b0 + n] = make_double2(fma(mel, e, diag), 0.0);
      }
      wave_sync();  // mv is rewritten by the next configuration
    }
  }
}

// O_k of 16 configurations per batch: g_l and g_h as products, then the K outputs with
// threads over the live parameters, each index pair used for the whole batch.
// Bound: writing B K values.  3e5 configurations, N = 50, H = 29, float32: 0.80 -> 0.54 ms
// (1.83 GB).
template <typename OutT>
__global__ __launch_bounds__(AB_NT, 4) void k_ar_grad16(ar_net d, const uint64_t* __restrict__ s, int64_t B,
                                                     const int2* __restrict__ idx, int64_t r1, int64_t r2, int64_t r3,
                                                     int64_t K, OutT* __restrict__ O) {
  extern __shared__ double lds[];
  const ar_lds L = ar_lds_at(d, lds, d.Hs);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
  ar_load(d, L);
  for (int64_t b0 = (int64_t)blockIdx.x * AB; b0 < B; b0 += (int64_t)gridDim.x * AB) {
    __syncthreads();
    ar_hidden16<false>(d, L, s, b0, B);
    for (int nt = wave; nt < d.NT2; nt += AB_WAVES) {
      const doublex4 l = ar_logits16(d, L, nt, li, lk);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double x = ar_bit(d, L, lk + 4 * r, min(16 * nt + li, d.N - 1));
        L.l[(lk + 4 * r) * d.Ns + 16 * nt + li] = x - 1.0 / (1.0 + m64::fexp(-l[r]));
      }
    }
    __syncthreads();
    for (int nt = wave; nt < d.NT1; nt += AB_WAVES) {
      doublex4 acc = doublex4{0.0, 0.0, 0.0, 0.0};
      for (int i0 = 0; i0 < d.N; i0 += 4)  // outputs past N: W2 is 0
        acc = mfma64(L.l[li * d.Ns + i0 + lk], L.W2[(16 * nt + li) * d.Ns + i0 + lk], acc);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int e = (lk + 4 * r) * d.Hs + 16 * nt + li;
        L.x2[e] = L.a[e] > 0.0 ? 0.5 * acc[r] : 0.0;
      }
    }
    __syncthreads();
    const int nb = (int)min((int64_t)AB, B - b0);
    for (int64_t j = threadIdx.x; j < K; j += AB_NT) {
      const int2 pr = idx[j];
      const int region = j < r1 ? 0 : j < r2 ? 1 : j < r3 ? 2 : 3;
      OutT* o = O + b0 * K + j;
      for (int n = 0; n < nb; ++n, o += K) {
        double v;
        if (region == 0)
          v = get_bit(L.bits + n * d.W, pr.y) ? L.x2[n * d.Hs + pr.x] : 0.0;
        else if (region == 1)
          v = L.x2[n * d.Hs + pr.x];
        else if (region == 2)
          v = 0.5 * L.l[n * d.Ns + pr.x] * fmax(L.a[n * d.Hs + pr.y], 0.0);
        else
          v = 0.5 * L.l[n * d.Ns + pr.x];
        if constexpr (std::is_same<OutT, double2>::value)
          *o = make_double2(v, 0.0);
        else if constexpr (std::is_same<OutT, float2>::value)
          *o = make_float2((float)v, 0.0f);
        else
          *o = (OutT)v;
      }
    }
  }
}

// the padded weights of ar_net, hidden units by position
__global__ void k_ar_pad(ar_net d, const double* __restrict__ W1mT, const double* __restrict__ W2m,
                         const double* __restrict__ b1, const double* __restrict__ b2, const int* __restrict__ perm,
                         double* __restrict__ pad) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  const int n1 = d.n4() * d.Hs, n2 = n1 + 16 * d.NT1 * d.Ns;
  if (e >= d.w_doubles()) return;
  double v = 0.0;
  if (e < n1) {
    const int i = e / d.Hs, k = e - i * d.Hs;
    if (i < d.N && k < d.H) v = W1mT[(int64_t)i * d.H + perm[k]];
  } else if (e < n2) {
    const int k = (e - n1) / d.Ns, i = (e - n1) - k * d.Ns;
    if (i < d.N && k < d.H) v = W2m[(int64_t)i * d.H + perm[k]];
  } else if (e < n2 + d.Hs) {
    if (e - n2 < d.H) v = b1[perm[e - n2]];
  } else if (e - n2 - d.Hs < d.N) {
    v = b2[e - n2 - d.Hs];
  }
  pad[e] = v;
}

// compact live parameters -> dense masked layout [W1 (H x N) | b1 | W2 (N x H) | b2]
__global__ void k_ar_scatter(const double2* __restrict__ theta, const int2* __restrict__ idx, int64_t r1, int64_t r2,
                             int64_t r3, int64_t K, int N, int H, double* __restrict__ dense) {
  const int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (j >= K) return;
  const int2 pr = idx[j];
  const int64_t HN = (int64_t)H * N;
  int64_t at;
  if (j < r1)
    at = (int64_t)pr.x * N + pr.y;
  else if (j < r2)
    at = HN + pr.x;
  else if (j < r3)
    at = HN + H + (int64_t)pr.x * H + pr.y;
  else
    at = 2 * HN + H + pr.x;
  dense[at] = theta[j].x;
}

__global__ void k_ar_transpose(const double* __restrict__ W2m, int N, int H, double* __restrict__ W2t) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= (int64_t)N * H) return;
  const int i = (int)(e / H), k = (int)(e % H);
  W2t[(int64_t)k * N + i] = W2m[e];
}

__global__ void k_ar_half(const double* __restrict__ lq, int64_t B, double2* __restrict__ out) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e < B) out[e] = make_double2(0.5 * lq[e], 0.0);
}

struct ar_ptrs {
  const double *W1mT, *W2m, *b1, *b2;
};

ar_ptrs ptrs(const vmc_model* m) {
  const vmc_made* md = m->made;
  const int64_t HN = (int64_t)m->Nh * m->N;
  return ar_ptrs{md->W1mT, md->W2m, md->params + HN, md->params + 2 * HN + m->Nh};
}

constexpr size_t kArLdsMax = 64 * 1024;

// Rows of 16 NT1 + 4 and 32 m + 20 doubles: 16 rows read at once start 8 words (Hs) or
// 40 words (Ns) apart in the 64 banks.
ar_net net_of(const vmc_model* m) {
  ar_net d;
  d.N = m->N;
  d.H = m->Nh;
  d.W = m->W;
  d.NT1 = (m->Nh + 15) / 16;
  d.NT2 = (m->N + 15) / 16;
  d.Hs = 16 * d.NT1 + 4;
  d.Ns = (16 * d.NT2 + 11) / 32 * 32 + 20;
  d.pm = std::min(m->Nh, m->N - 1);
  d.pad = m->ar_pad;
  d.mst = m->ar_perm + m->Nh;
  return d;
}

// LDS bytes of the 16-configuration kernels, or 0 where they do not apply: the product of N
// factors in [1, 2] has to stay in range, and the padded weights have to fit beside a batch.
constexpr size_t kArBatchLds = 158 * 1024;
size_t batch_lds(const ar_net& d, int x2, size_t extra = 0) {
  const size_t b = sizeof(double) * ar_lds_doubles(d, x2) + extra;
  return d.N <= 512 && b <= kArBatchLds ? b : 0;
}

unsigned batch_groups(vmc_ctx* ctx, int64_t B, size_t lds) {
  const int64_t per_cu = std::max<int64_t>(1, std::min<int64_t>(8, (int64_t)(160 * 1024) / (int64_t)lds));
  return (unsigned)std::min<int64_t>((B + AB - 1) / AB, cu_count(ctx) * per_cu);
}

template <typename Kern>
void batch_allow(Kern k, size_t lds) {
  if (lds > 64 * 1024) VMC_HIP(hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
}

void* ar_alloc(size_t bytes) {
  void* p = nullptr;
  if (hipMalloc(&p, bytes) != hipSuccess) {
    (void)hipGetLastError();
    throw vmc_error{VMC_ERR_OOM, "device allocation failed"};
  }
  return p;
}

}  // namespace

void ar_init(vmc_model* m) {
  const int N = m->N, H = m->Nh;
  std::vector<int2> idx;
  idx.reserve((size_t)m->K);
  auto deg = [&](int k) { return k % (N - 1) + 1; };
  for (int k = 0; k < H; ++k)
    for (int d = 0; d < deg(k); ++d) idx.push_back(make_int2(k, d));
  m->ar_r1 = (int64_t)idx.size();
  for (int k = 0; k < H; ++k) idx.push_back(make_int2(k, 0));
  m->ar_r2 = (int64_t)idx.size();
  for (int i = 0; i < N; ++i)
    for (int k = 0; k < H; ++k)
      if (deg(k) <= i) idx.push_back(make_int2(i, k));
  m->ar_r3 = (int64_t)idx.size();
  for (int i = 0; i < N; ++i) idx.push_back(make_int2(i, 0));
  if ((int64_t)idx.size() != m->K) throw vmc_error{VMC_ERR_INVALID_ARG, "internal: live parameter count mismatch"};
  vmc_ctx* ctx = m->ctx;
  vmc_made* md = nullptr;
  if (vmc_made_create(ctx, N, H, &md) != VMC_OK) throw vmc_error{VMC_ERR_OOM, vmc_last_error(ctx)};
  m->made = md;
  m->ar_idx = (int2*)ar_alloc(sizeof(int2) * idx.size());
  m->ar_w2t = (double*)ar_alloc(sizeof(double) * (size_t)N * H);
  // hidden units by degree: position -> unit, first position per degree, index pairs by position
  std::vector<int> perm, mst, at(H);
  mix_made_layout(N, H, perm, mst);
  for (int q = 0; q < H; ++q) at[perm[q]] = q;
  std::vector<int2> idxp = idx;
  for (int64_t j = 0; j < m->ar_r3; ++j) (j < m->ar_r2 ? idxp[j].x : idxp[j].y) = at[j < m->ar_r2 ? idx[j].x : idx[j].y];
  perm.insert(perm.end(), mst.begin(), mst.end());
  m->ar_idxp = (int2*)ar_alloc(sizeof(int2) * idxp.size());
  m->ar_perm = (int*)ar_alloc(sizeof(int) * perm.size());
  m->ar_pad = (double*)ar_alloc(sizeof(double) * net_of(m).w_doubles());
  VMC_HIP(hipMemcpyAsync(m->ar_idxp, idxp.data(), sizeof(int2) * idxp.size(), hipMemcpyHostToDevice, ctx->stream));
  VMC_HIP(hipMemcpyAsync(m->ar_perm, perm.data(), sizeof(int) * perm.size(), hipMemcpyHostToDevice, ctx->stream));
  VMC_HIP(hipMemcpyAsync(m->ar_idx, idx.data(), sizeof(int2) * idx.size(), hipMemcpyHostToDevice, ctx->stream));
  VMC_HIP(hipStreamSynchronize(ctx->stream));
  ar_set_params(m);
}

void ar_free(vmc_model* m) {
  if (m->ar_idx) (void)hipFree(m->ar_idx);
  if (m->ar_w2t) (void)hipFree(m->ar_w2t);
  if (m->ar_idxp) (void)hipFree(m->ar_idxp);
  if (m->ar_perm) (void)hipFree(m->ar_perm);
  if (m->ar_pad) (void)hipFree(m->ar_pad);
  m->ar_idxp = nullptr;
  m->ar_perm = nullptr;
  m->ar_pad = nullptr;
  if (m->made) (void)vmc_made_destroy(m->made);
  m->ar_idx = nullptr;
  m->ar_w2t = nullptr;
  m->made = nullptr;
}

void ar_set_params(vmc_model* m) {
  vmc_made* md = m->made;
  hipStream_t st = m->ctx->stream;
  VMC_HIP(hipMemsetAsync(md->params, 0, sizeof(double) * md->P, st));
  k_ar_scatter<<<grid_for(m->K, 256), 256, 0, st>>>(m->params, m->ar_idx, m->ar_r1, m->ar_r2, m->ar_r3, m->K, m->N,
                                                    m->Nh, md->params);
  VMC_HIP(hipGetLastError());
  made_refresh(md);
  const int64_t n = (int64_t)m->N * m->Nh;
  k_ar_transpose<<<grid_for(n, 256), 256, 0, st>>>(md->W2m, m->N, m->Nh, m->ar_w2t);
  const ar_net d = net_of(m);
  const ar_ptrs p = ptrs(m);
  k_ar_pad<<<grid_for(d.w_doubles(), 256), 256, 0, st>>>(d, p.W1mT, p.W2m, p.b1, p.b2, m->ar_perm, m->ar_pad);
  VMC_HIP(hipGetLastError());
}

void ar_log_psi(vmc_model* m, const uint64_t* s, int64_t B, double2* out) {
  const ar_net d = net_of(m);
  const size_t lw = sizeof(double) * (d.w_doubles() + (d.N + 2) / 2 + (size_t)AB_WAVES * AB * (d.W + d.Hs));
  // few configurations: a group each (a batch's wave goes through all sites on its own while
  // most of the chip idles).  Both cost the same near 1 000 + 50 N configurations up to 160 sites,
  // where the general kernel's time per configuration stops growing with N: 10 sites, 8 units,
  // 1 024 configurations 16.4 against 17.1 us; 50, 29: 1 024 18 against 26, 8 192 35 against 26;
  // 128, 32: 4 096 31 against 38, 12 288 58 against 39
  const bool many = B >= 1024 + 48 * (int64_t)std::min(d.N, 160);
  if (many && d.N <= 512 && lw <= kArBatchLds) {
    batch_allow(k_ar_log_psi16, lw);
    k_ar_log_psi16<<<batch_groups(m->ctx, (B + AB_WAVES - 1) / AB_WAVES, lw), AB_NT, lw, m->ctx->stream>>>(d, s, B, out);
    VMC_HIP(hipGetLastError());
    return;
  }
  const ar_ptrs p = ptrs(m);
  const size_t lds = sizeof(double) * (2 * (size_t)m->N + 2 * (size_t)m->Nh);
  for (int64_t b0 = 0; b0 < B; b0 += INT32_MAX) {
    const int64_t nb = std::min<int64_t>(INT32_MAX, B - b0);
    k_ar_log_psi<<<(unsigned)nb, AR_NT, lds, m->ctx->stream>>>(s + b0 * m->W, m->N, m->Nh, m->W, p.W1mT, m->ar_w2t,
                                                              p.b1, p.b2, out + b0);
    VMC_HIP(hipGetLastError());
  }
}

void ar_local_energy(vmc_model* m, vmc_ham* H, const uint64_t* s, int64_t B, double2* eloc) {
  const ar_ptrs p = ptrs(m);
  const ar_net d = net_of(m);
  // the Heisenberg move lists of the waves follow the batch
  const size_t extra = sizeof(int) * (H->kind == HAM_HEIS ? (size_t)AB_WAVES * H->n_bonds : 0);
  // few configurations of a small network: a group each, without the batch's barriers and padded
  // weights (10 sites, 8 units, 512 configurations, exchanges 21 against 24 us, 2 048 27 against 24;
  // 3 sites, one unit, 1 024 18.5 against 23 us)
  const bool few = B <= 2048 && B * m->K <= 1 << 16 && (m->K < 64 || (m->K < 160 && B >= 16));
  if (const size_t lb = few ? 0 : batch_lds(d, d.Ns, extra)) {
    batch_allow(k_ar_eloc16, lb);
    k_ar_eloc16<<<batch_groups(m->ctx, B, lb), AB_NT, lb, m->ctx->stream>>>(d, s, B, H->kind, H->J, H->h, H->bonds,
                                                                           H->n_bonds, eloc);
    VMC_HIP(hipGetLastError());
    return;
  }
  const size_t lds = sizeof(double) * (3 * (size_t)m->N + 2 * (size_t)m->Nh) + sizeof(int) * (size_t)H->n_bonds;
  VMC_REQUIRE(lds <= kArLdsMax, "network too large for the per-configuration local-energy tile");
  const int QH = (m->Nh + 63) / 64;
  for (int64_t b0 = 0; b0 < B; b0 += INT32_MAX) {
    const int64_t nb = std::min<int64_t>(INT32_MAX, B - b0);
#define AR_ELOC(Q)                                                                                                 \
  k_ar_eloc<Q><<<(unsigned)nb, AR_NT, lds, m->ctx->stream>>>(s + b0 * m->W, m->N, m->Nh, m->W, p.W1mT, m->ar_w2t, \
                                                             p.b1, p.b2, H->kind, H->J, H->h, H->bonds, H->n_bonds, \
                                                             eloc + b0)
    if (QH <= 1)
      AR_ELOC(1);
    else if (QH <= 2)
      AR_ELOC(2);
    else if (QH <= 4)
      AR_ELOC(4);
    else if (QH <= 8)
      AR_ELOC(8);
    else
      AR_ELOC(16);
#undef AR_ELOC
    VMC_HIP(hipGetLastError());
  }
}

void ar_grad(vmc_model* m, const uint64_t* s, int64_t B, void* O, int dtype) {
  const ar_ptrs p = ptrs(m);
  const ar_net d = net_of(m);
  const size_t lb = batch_lds(d, d.Hs);
  const size_t lw = sizeof(double) * (2 * (size_t)m->N * m->Nh + (size_t)AR_WAVES * (2 * (size_t)m->N + 2 * m->Nh));
  // a configuration per wave where the network fits it and does not fill the 16 x 16 operands
  // (fewer than 128 parameters: 10 sites, 8 units, 512 configurations 18 against 21 us, 131 072 88
  // against 104), has too many sites for the padded weights (350 sites, 3 units, 8 192 105 against
  // the general kernel's 240 us), is small and comes with few configurations (30 sites, 20 units,
  // 512 22.6 against 24 us; one alone 21 against 19) or writes long complex128 rows, which a
  // wave finishes on its own (50 sites, 29 units, 32 768 185 against 198 us; 64 sites, 50 units
  // 466 against 392)
  const bool wide = dtype == VMC_DT_C128 && B >= 16384 && m->K >= 512 && m->K < 2048;
  if (lw <= kArLdsMax && ((!lb && B >= AR_WAVES) || m->K < 128 || (m->K < 1024 && B >= 16 && B <= 512) || wide)) {
    const int64_t per_cu = std::max<int64_t>(1, std::min<int64_t>(8, (int64_t)(160 * 1024) / (int64_t)lw));
    const unsigned g = (unsigned)std::min<int64_t>((B + AR_WAVES - 1) / AR_WAVES, cu_count(m->ctx) * per_cu);
    auto run = [&](auto* o) {
      using T = std::remove_pointer_t<decltype(o)>;
      k_ar_grad_w<T><<<g, AR_NT, lw, m->ctx->stream>>>(s, B, m->N, m->Nh, m->W, p.W1mT, m->ar_w2t, p.b1, p.b2,
                                                       m->ar_idx, m->ar_r1, m->ar_r2, m->ar_r3, m->K, o);
      VMC_HIP(hipGetLastError());
    };
    if (dtype == VMC_DT_C128)
      run((double2*)O);
    else if (dtype == VMC_DT_C64)
      run((float2*)O);
    else if (dtype == VMC_DT_F64)
      run((double*)O);
    else
      run((float*)O);
    return;
  }
  if (lb) {
    auto run = [&](auto* o) {
      using T = std::remove_pointer_t<decltype(o)>;
      batch_allow(k_ar_grad16<T>, lb);
      k_ar_grad16<T><<<batch_groups(m->ctx, B, lb), AB_NT, lb, m->ctx->stream>>>(d, s, B, m->ar_idxp, m->ar_r1, m->ar_r2,
                                                                                 m->ar_r3, m->K, o);
      VMC_HIP(hipGetLastError());
    };
    if (dtype == VMC_DT_C128)
      run((double2*)O);
    else if (dtype == VMC_DT_C64)
      run((float2*)O);
    else if (dtype == VMC_DT_F64)
      run((double*)O);
    else
      run((float*)O);
    return;
  }
  const size_t per = sizeof(double) * (2 * (size_t)m->N + 3 * (size_t)m->Nh);
  const int sb = 4 * per <= kArLdsMax ? 4 : 1;
  VMC_REQUIRE(per <= kArLdsMax, "network too large for the per-configuration gradient tile");
  const int64_t groups = (B + sb - 1) / sb;
  VMC_REQUIRE(groups <= INT32_MAX, "too many configurations for one launch");
  hipStream_t st = m->ctx->stream;
#define AR_GRAD(S, T)                                                                                           \
  k_ar_grad<S, T><<<(unsigned)groups, AR_NT, S * per, st>>>(s, B, m->N, m->Nh, m->W, p.W1mT, m->ar_w2t, p.W2m, \
                                                            p.b1, p.b2, m->ar_idx, m->ar_r1, m->ar_r2, m->ar_r3, \
                                                            m->K, (T*)O)
  if (dtype == VMC_DT_C128) {
    if (sb == 4)
      AR_GRAD(4, double2);
    else
      AR_GRAD(1, double2);
  } else if (dtype == VMC_DT_C64) {
    if (sb == 4)
      AR_GRAD(4, float2);
    else
      AR_GRAD(1, float2);
  } else if (dtype == VMC_DT_F64) {
    if (sb == 4)
      AR_GRAD(4, double);
    else
      AR_GRAD(1, double);
  } else {
    if (sb == 4)
      AR_GRAD(4, float);
    else
      AR_GRAD(1, float);
  }
#undef AR_GRAD
  VMC_HIP(hipGetLastError());
}

void ar_sample(vmc_sampler* S, int64_t B, uint64_t* s_out, double2* logpsi_out) {
  vmc_model* m = S->model;
  vmc_ctx* ctx = S->ctx;
  VMC_REQUIRE(B <= INT32_MAX, "at most 2^31 - 1 direct samples per call");
  double* lq = nullptr;
  if (logpsi_out) {
    ws_reserve(ctx, ws_round(sizeof(double) * B));
    lq = (double*)ws_take(ctx, sizeof(double) * B);
  }
  made_sample_impl(m->made, B, S->opts.seed, S->t, s_out, lq);
  if (logpsi_out) {
    k_ar_half<<<grid_for(B, 256), 256, 0, ctx->stream>>>(lq, B, logpsi_out);
    VMC_HIP(hipGetLastError());
  }
  S->t += 1;
}
