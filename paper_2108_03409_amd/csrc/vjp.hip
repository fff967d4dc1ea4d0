// Vector-Jacobian product of log psi for reverse-mode autodiff:
//   out_k = sum_n g_n conj(O_nk),   O_nk = d log psi(s_n) / d theta_k,
// the backward of a holomorphic map in the conjugate-Wirtinger convention.
// Nothing of the forward pass is kept; and O itself is never stored:
//
//  RBM: with U_nj = g_n conj(tanh theta_nj) and sigma_ni = +-1,
//         out_W[j][i] = sum_n U_nj sigma_ni,  out_b[j] = sum_n U_nj,
//         out_a[i]    = sum_n g_n sigma_ni,
//       i.e. one product [N_h + 1 rows: U and g] x [N + 1 columns: sigma and
//       1] over the samples, split over sample ranges, the slices added in a
//       fixed order.  Up to 128 sites theta, U and the product stay in one
//       kernel's registers (k_vjp_rbm); beyond, theta and U go through memory
//       and two real float64 matrix-core GEMMs (Re and Im of U).
//  CNN: the gradient kernel recomputes both layers per sample and each
//       work-group accumulates g_n conj(O_n) over its samples into one row of
//       partial sums, which a second kernel adds in a fixed order.
//
// Scratch: the context's workspace (vmc_log_psi_vjp), or, for callers that
// cannot allocate, a fixed device array owned by this file
// (vmc_log_psi_vjp_noalloc).  Either way the work is chunked over samples to
// fit the scratch it is given.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>

#include "internal.h"

using namespace dev;

namespace {

constexpr int kSplit = 32;     // sample ranges of the RBM product
constexpr int kCnnGroups = 256;  // work-groups (partial rows) of the CNN product

typedef double doublex4 __attribute__((ext_vector_type(4)));

constexpr int kUnits = 16;     // units of a work-group of k_vjp_rbm
constexpr int kBatch = 64;     // samples of a step of it, 16 per wave
constexpr int kFusedTiles = 8; // at most 16 * 8 sites

__device__ __forceinline__ double sign_of(uint64_t w, int i) {  // +1 where bit i is set, else -1
  return __hiloint2double((int)(0xBFF00000u ^ ((uint32_t)(w >> i) << 31)), 0);
}

// part[z][j][i] = sum over the samples of range z of U_nj sigma_ni (i < N) and U_nj (i = N),
// for 16 units j (N_h stands for g itself) and up to 16 NT sites.
// A wave takes 16 samples at a time: theta = b + sigma W is one product on the float64
// matrix cores (rows samples, columns units), and since register r of lane l then holds
// sample l / 16 + 4 r of unit l % 16, U = g conj(tanh theta) is at once the left operand of
// the second product (rows units, reduction over samples, columns sites): nothing but the
// spins and g is read per sample, the weights of the 16 units stand in LDS.
// Bound: the float64 matrix cores with the tanh beside them (64 MFMAs and four tanh per
// lane a step at 64 sites).  N = 64, N_h = 256, 16 384 samples: the whole call 190 -> 85 us
// (theta, U and sigma through memory and two GEMMs before).
template <int NT>
__global__ __launch_bounds__(256, 2) void k_vjp_rbm(const double2* __restrict__ params, const double2* __restrict__ Wt,
                                                    const uint64_t* __restrict__ s, const double2* __restrict__ g,
                                                    int64_t B, int N, int W, int Nh, double2* __restrict__ part) {
  constexpr int NW = (NT + 3) / 4;            // words of a configuration (those past W read as 0)
  __shared__ double2 wl[NT * 16 * kUnits];    // [site][unit]; the slice's entries [unit][site] at the end
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, li = lane & 15, lk = lane >> 4;
  const int u0 = blockIdx.x * kUnits, unit = u0 + li;
  for (int e = tid; e < NT * 16 * kUnits; e += 256) {
    const int i = e / kUnits, j = u0 + e % kUnits;
    wl[e] = make_double2(0.0, 0.0);
    if (i < N && j < Nh) wl[e] = Wt[(int64_t)i * Nh + j];
  }
  __syncthreads();
  double2 bj = make_double2(0.0, 0.0);
  if (unit < Nh) bj = params[N + unit];
  const int64_t nb = (B + kBatch - 1) / kBatch;
  const int64_t t0 = nb * blockIdx.y / gridDim.y, t1 = nb * (blockIdx.y + 1) / gridDim.y;
  doublex4 cr[NT], ci[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) cr[t] = ci[t] = doublex4{0.0, 0.0, 0.0, 0.0};
  double2 ones = make_double2(0.0, 0.0);
  for (int64_t bt = t0; bt < t1; ++bt) {
    const int64_t n0 = bt * kBatch + 16 * wv;
    uint64_t wa[NW], wb[4][NW];  // spins of sample li (theta) and of samples lk + 4 r (product)
    double2 gr[4];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      wa[w] = 0ull;
      if (n0 + li < B && w < W) wa[w] = s[(n0 + li) * W + w];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t n = n0 + lk + 4 * r;
      gr[r] = make_double2(0.0, 0.0);
      if (n < B) gr[r] = g[n];
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        wb[r][w] = 0ull;
        if (n < B && w < W) wb[r][w] = s[n * W + w];
      }
    }
    doublex4 tr = doublex4{bj.x, bj.x, bj.x, bj.x}, ti = doublex4{bj.y, bj.y, bj.y, bj.y};
#pragma unroll
    for (int w = 0; w < NW; ++w)
#pragma unroll 4
      for (int q = 16 * w; q < (4 * NT < 16 * w + 16 ? 4 * NT : 16 * w + 16); ++q) {
        const int i = 4 * q + lk;
        const double a = sign_of(wa[w], i & 63);
        const double2 v = wl[i * kUnits + li];
        tr = __builtin_amdgcn_mfma_f64_16x16x4f64(a, v.x, tr, 0, 0, 0);
        ti = __builtin_amdgcn_mfma_f64_16x16x4f64(a, v.y, ti, 0, 0, 0);
      }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      double2 u = make_double2(0.0, 0.0);
      if (n0 + lk + 4 * r < B && unit < Nh) u = cmul(gr[r], cconj(ctanh(make_double2(tr[r], ti[r]))));
      if (unit == Nh) u = gr[r];
      ones = cadd(ones, u);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const double sg = sign_of(wb[r][t / 4], (16 * t + li) & 63);
        cr[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(u.x, sg, cr[t], 0, 0, 0);
        ci[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(u.y, sg, ci[t], 0, 0, 0);
      }
    }
  }
  // the four waves' sums, in wave order
  double2* out = part + (int64_t)blockIdx.y * (Nh + 1) * (N + 1);
  ones.x += __shfl_xor(ones.x, 16, 64);
  ones.y += __shfl_xor(ones.y, 16, 64);
  ones.x += __shfl_xor(ones.x, 32, 64);
  ones.y += __shfl_xor(ones.y, 32, 64);
  __shared__ double2 os[4][kUnits];
  if (lk == 0) os[wv][li] = ones;
  for (int w = 0; w < 4; ++w) {
    __syncthreads();
    if (wv == w) {
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          double2& c = wl[(lk + 4 * r) * (16 * NT) + 16 * t + li];
          c = w == 0 ? make_double2(cr[t][r], ci[t][r]) : make_double2(c.x + cr[t][r], c.y + ci[t][r]);
        }
    }
  }
  __syncthreads();
  for (int e = tid; e < NT * 16 * kUnits; e += 256) {
    const int j = e / (16 * NT), i = e % (16 * NT);
    if (i < N && u0 + j <= Nh) out[(int64_t)(u0 + j) * (N + 1) + i] = wl[e];
  }
  if (tid < kUnits && u0 + tid <= Nh)
    out[(int64_t)(u0 + tid) * (N + 1) + N] = cadd(cadd(os[0][tid], os[1][tid]), cadd(os[2][tid], os[3][tid]));
}

// entry of the [N_h + 1][N + 1] product that is output e
__device__ __forceinline__ int64_t vjp_entry(int64_t e, int N, int Nh) {
  if (e < N) return (int64_t)Nh * (N + 1) + e;            // a_i: row of g
  if (e < N + Nh) return (e - N) * (N + 1) + N;           // b_j: column of ones
  const int64_t r = e - N - Nh;                           // W[j][i]
  return (r / N) * (N + 1) + r % N;
}

// out from the slices of k_vjp_rbm: wave w of a group adds slices w, w + 4, ... of 64
// outputs, the four sums in wave order
__global__ __launch_bounds__(256) void k_vjp_rbm_sum(const double2* __restrict__ part, int N, int Nh, int nz,
                                                     double2* __restrict__ out) {
  __shared__ double2 red[4][64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t e = blockIdx.x * 64ll + lane, K = (int64_t)N + Nh + (int64_t)Nh * N;
  const int64_t slice = (int64_t)(Nh + 1) * (N + 1);
  double2 acc = make_double2(0.0, 0.0);
  if (e < K) {
    const double2* p = part + vjp_entry(e, N, Nh);
#pragma unroll 8
    for (int z = wv; z < nz; z += 4) acc = cadd(acc, p[z * slice]);
  }
  red[wv][lane] = acc;
  __syncthreads();
  if (wv == 0 && e < K) out[e] = cadd(cadd(red[0][lane], red[1][lane]), cadd(red[2][lane], red[3][lane]));
}

// U'[n][j] = g_n conj(tanh theta_nj) (j < N_h), U'[n][N_h] = g_n; S'[n][i] = sigma_ni (i < N), S'[n][N] = 1.
__global__ __launch_bounds__(256) void k_vjp_rbm_prep(const double2* __restrict__ theta, const uint64_t* __restrict__ s,
                                                      const double2* __restrict__ g, int64_t B, int N, int W, int Nh,
                                                      double2* __restrict__ U, double* __restrict__ Sg) {
  const int64_t n = blockIdx.x;
  if (n >= B) return;
  const double2 gn = g[n];
  const uint64_t* sn = s + n * W;
  for (int j = threadIdx.x; j <= Nh; j += 256)
    U[n * (Nh + 1) + j] = j < Nh ? cmul(gn, cconj(ctanh(theta[n * Nh + j]))) : gn;
  for (int i = threadIdx.x; i <= N; i += 256) Sg[n * (N + 1) + i] = i < N ? (get_bit(sn, i) ? 1.0 : -1.0) : 1.0;
}

// out from the kSplit slices of C_re, C_im ([N_h + 1][N + 1] each): fixed order
__global__ void k_vjp_rbm_out(const double* __restrict__ Cre, const double* __restrict__ Cim, int N, int Nh,
                              int64_t slice, int nsplit, double2* __restrict__ out) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t K = (int64_t)N + Nh + (int64_t)Nh * N;
  if (e >= K) return;
  const int64_t c = vjp_entry(e, N, Nh);
  double re = 0.0, im = 0.0;
  for (int z = 0; z < nsplit; ++z) {
    re += Cre[z * slice + c];
    im += Cim[z * slice + c];
  }
  out[e] = make_double2(re, im);
}

__global__ void k_zero2(double2* __restrict__ out, int64_t K) {
  const int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (k < K) out[k] = make_double2(0.0, 0.0);
}

__global__ void k_vjp_rows(const double2* __restrict__ part, int rows, int64_t K, double2* __restrict__ out) {
  const int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (k >= K) return;
  double2 acc = make_double2(0.0, 0.0);
  for (int q = 0; q < rows; ++q) acc = cadd(acc, part[(int64_t)q * K + k]);
  out[k] = acc;
}

// bytes of the fixed part of the RBM scratch, and per sample of a chunk
size_t rbm_fixed_bytes(const vmc_model* m) {
  return ws_round(sizeof(double) * 2 * (size_t)kSplit * (m->Nh + 1) * (m->N + 1));
}
size_t rbm_per_sample_bytes(const vmc_model* m) {
  return sizeof(double2) * (size_t)m->Nh + sizeof(double2) * (m->Nh + 1) + sizeof(double) * (m->N + 1);
}

// the product in one kernel (N <= 128): sample ranges for one round of the groups that
// the registers leave a compute unit (three of 168 at up to 64 sites, then two), as many
// as the scratch holds slices
void vjp_rbm_fused(vmc_model* m, const uint64_t* s, int64_t B, const double2* g, double2* out, char* scratch,
                   size_t bytes) {
  vmc_ctx* ctx = m->ctx;
  const int N = m->N, Nh = m->Nh, ub = Nh / kUnits + 1;
  const size_t slice = sizeof(double2) * (size_t)(Nh + 1) * (N + 1);
  const int64_t groups = (N <= 64 ? 3 : 2) * (int64_t)cu_count(ctx);
  const int64_t nz = std::max<int64_t>(
      1, std::min<int64_t>({groups / ub, (B + kBatch - 1) / kBatch, (int64_t)(bytes / slice)}));
  double2* part = (double2*)scratch;
  const dim3 grid(ub, (unsigned)nz);
  switch ((N + 15) / 16) {
#define CASE(T)                                                                                                 \
  case T:                                                                                                       \
    k_vjp_rbm<T><<<grid, 256, 0, ctx->stream>>>(m->params, m->Wt, s, g, B, N, m->W, Nh, part);                  \
    break
    CASE(1);
    CASE(2);
    CASE(3);
    CASE(4);
    CASE(5);
    CASE(6);
    CASE(7);
    CASE(8);
#undef CASE
    default: throw vmc_error{VMC_ERR_UNSUPPORTED, "internal: more than 128 sites"};
  }
  VMC_HIP(hipGetLastError());
  k_vjp_rbm_sum<<<(unsigned)((m->K + 63) / 64), 256, 0, ctx->stream>>>(part, N, Nh, (int)nz, out);
  VMC_HIP(hipGetLastError());
}

void vjp_rbm(vmc_model* m, const uint64_t* s, int64_t B, const double2* g, double2* out, char* scratch,
             size_t bytes) {
  vmc_ctx* ctx = m->ctx;
  const int N = m->N, Nh = m->Nh;
  if (N <= 16 * kFusedTiles) return vjp_rbm_fused(m, s, B, g, out, scratch, bytes);
  const size_t fixed = rbm_fixed_bytes(m);
  const int64_t chunk =
      std::min<int64_t>(B, (int64_t)((bytes - fixed - 3 * 256) / rbm_per_sample_bytes(m)));
  const int64_t slice = (int64_t)(Nh + 1) * (N + 1);
  double* Cre = (double*)scratch;
  double* Cim = Cre + (size_t)kSplit * slice;
  char* p = scratch + fixed;
  double2* theta = (double2*)p;
  p += ws_round(sizeof(double2) * (size_t)chunk * Nh);
  double2* U = (double2*)p;
  p += ws_round(sizeof(double2) * (size_t)chunk * (Nh + 1));
  double* Sg = (double*)p;
  for (int64_t b0 = 0; b0 < B; b0 += chunk) {
    const int64_t nb = std::min(chunk, B - b0);
    rbm_theta(m, s + b0 * m->W, nb, theta);
    k_vjp_rbm_prep<<<(unsigned)nb, 256, 0, ctx->stream>>>(theta, s + b0 * m->W, g + b0, nb, N, m->W, Nh, U, Sg);
    VMC_HIP(hipGetLastError());
    const int64_t kc = (nb + kSplit - 1) / kSplit;
    const double beta = b0 == 0 ? 0.0 : 1.0;
    // C[j][i] (+)= sum_n A(j, n) Sg[n][i], A = Re U' / Im U' read in place (stride 2 doubles)
    dgemm_args re{(const double*)U, 2, 2 * (int64_t)(Nh + 1), Sg, N + 1, 1, Cre, N + 1, Nh + 1, N + 1, nb, beta,
                  kc, slice};
    dgemm_args im = re;
    im.A = (const double*)U + 1;
    im.C = Cim;
    dgemm(ctx, re, kSplit);
    dgemm(ctx, im, kSplit);
  }
  const int64_t K = m->K;
  k_vjp_rbm_out<<<grid_for(K, 256), 256, 0, ctx->stream>>>(Cre, Cim, N, Nh, slice, kSplit, out);
  VMC_HIP(hipGetLastError());
}

void vjp_cnn(vmc_model* m, const uint64_t* s, int64_t B, const double2* g, double2* out, char* scratch,
             size_t bytes) {
  vmc_ctx* ctx = m->ctx;
  const int64_t K = m->K;
  const int groups = (int)std::min<int64_t>({B, (int64_t)kCnnGroups, (int64_t)(bytes / (sizeof(double2) * K))});
  double2* part = (double2*)scratch;
  cnn_vjp_partial(m, s, B, g, groups, part);
  k_vjp_rows<<<grid_for(K, 256), 256, 0, ctx->stream>>>(part, groups, K, out);
  VMC_HIP(hipGetLastError());
}

void vjp_run(vmc_model* m, const uint64_t* s, int64_t B, const double2* g, double2* out, char* scratch,
             size_t bytes) {
  if (m->kind == MODEL_RBM)
    vjp_rbm(m, s, B, g, out, scratch, bytes);
  else
    vjp_cnn(m, s, B, g, out, scratch, bytes);
}

// the smallest scratch that lets a model run (one sample per chunk / one partial row)
size_t min_scratch(const vmc_model* m) {
  if (m->kind == MODEL_RBM) return rbm_fixed_bytes(m) + 3 * 256 + rbm_per_sample_bytes(m);
  return sizeof(double2) * (size_t)m->K;
}

// ---- fixed scratch for callers that cannot allocate ------------------------
constexpr size_t kNoAllocBytes = (size_t)32 << 20;  // 32 MiB per device
__device__ __align__(256) char scratch[kNoAllocBytes];

std::mutex g_scratch_mu;
void* g_scratch_ptr[64] = {};

// Device address of `scratch` on the current device, looked up once per device
// with that device current (each device holds its own copy of the array; in
// host code the array's name is only a stand-in, never a device address).
char* noalloc_scratch() {
  int dev = 0;
  VMC_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) throw vmc_error{VMC_ERR_UNSUPPORTED, "device index above 63"};
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    VMC_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    g_scratch_ptr[dev] = p;
  }
  return (char*)g_scratch_ptr[dev];
}

}  // namespace

void log_psi_vjp_impl(vmc_model* m, const uint64_t* s, int64_t B, const double2* g, double2* out) {
  vmc_ctx* ctx = m->ctx;
  if (B == 0) {
    k_zero2<<<grid_for(m->K, 256), 256, 0, ctx->stream>>>(out, m->K);
    VMC_HIP(hipGetLastError());
    return;
  }
  size_t bytes;
  if (m->kind == MODEL_RBM) {
    const int64_t chunk = std::min<int64_t>(B, 65536);
    bytes = rbm_fixed_bytes(m) + 3 * 256 + (size_t)chunk * rbm_per_sample_bytes(m);
  } else {
    bytes = sizeof(double2) * (size_t)std::min<int64_t>(B, kCnnGroups) * m->K;
  }
  bytes = ws_round(bytes);
  ws_reserve(ctx, bytes);
  char* ws = (char*)ws_take(ctx, bytes);
  vjp_run(m, s, B, g, out, ws, bytes);
}

void log_psi_vjp_noalloc_impl(vmc_model* m, const uint64_t* s, int64_t B, const double2* g, double2* out) {
  const size_t need = min_scratch(m);
  if (need > kNoAllocBytes)
    throw vmc_error{VMC_ERR_WORKSPACE, "model needs " + std::to_string(need) + " bytes of scratch; the fixed " +
                                           "no-allocation scratch holds " + std::to_string(kNoAllocBytes)};
  char* sc = noalloc_scratch();
  if (B == 0) {
    k_zero2<<<grid_for(m->K, 256), 256, 0, m->ctx->stream>>>(out, m->K);
    VMC_HIP(hipGetLastError());
    return;
  }
  vjp_run(m, s, B, g, out, sc, kNoAllocBytes);
}
