// S = X^H X in float64 on the matrix cores (complex128 / float64 log-derivatives):
//   S_rc = sum_n conj(X_nr) X_nc,  Re = sum (xr xr' + xi xi'),  Im = sum (xr xi' - xi xr'),
// four real products per complex term; real X (two samples per complex row) needs the
// real part only, two products.
//
// 64 x 64 tiles of the lower triangle, 2 x 2 waves of 32 x 32 each; 16 samples a stage in
// two LDS buffers, the next stage's loads in flight over the current one's products.
// Where the tiles leave compute units idle (small K, many samples) the samples are split
// over grid z and the partial tiles are added in order by a second kernel, which also
// projects, shifts and mirrors.
//
// Bound: the float64 matrix cores.  K = 404 real, 40 000 samples (the pairs of one
// half as many rows): 3.53 -> 0.39 ms; the vector kernel it replaces ran 32 x 32 tiles with
// 91 groups on 256 compute units.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "internal.h"

using namespace dev;

namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));

constexpr int HT = 64;   // tile
constexpr int HS = 16;   // samples per stage

struct h64_args {
  const double2* X;
  int64_t N, K;
  int64_t per;  // samples per split
  int mode;
  double nu, eps;
  double2* S;
  double2* diag;
  double* part;  // [split][tile][values of HT x HT]; nullptr: one split, written to S
  int ntiles;
};

__device__ __forceinline__ void h64_tile(int lin, int& tr, int& tc) {
  tr = (int)((sqrt(8.0 * (double)lin + 1.0) - 1.0) * 0.5);
  while ((tr + 1) * (tr + 2) / 2 <= lin) ++tr;
  while (tr * (tr + 1) / 2 > lin) --tr;
  tc = lin - tr * (tr + 1) / 2;
}

__device__ __forceinline__ void h64_put(const h64_args& a, int64_t r, int64_t c, double2 v) {
  if (r >= a.K || c > r) return;
  if (a.mode == VMC_SR_REAL) v.y = 0.0;
  if (a.mode == VMC_SR_IMAG) v.x = 0.0;  // i Im S
  if (r == c) {
    v = make_double2(v.x * (1.0 + a.nu) + a.eps, 0.0);
    a.diag[r] = v;
  }
  a.S[r * a.K + c] = v;
  if (r != c) a.S[c * a.K + r] = cconj(v);
}

template <bool REAL>
__global__ __launch_bounds__(256, 2) void k_herk64(h64_args a) {
  __shared__ double2 As[2][HS][HT + 1];
  __shared__ double2 Bs[2][HS][HT + 1];
  int tr, tc;
  h64_tile(blockIdx.x, tr, tc);
  const int64_t r0 = (int64_t)tr * HT, c0 = (int64_t)tc * HT;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave >> 1, wc = wave & 1, li = lane & 15, lk = lane >> 4;
  const int64_t n0 = (int64_t)blockIdx.y * a.per, n1 = min(a.N, n0 + a.per);
  doublex4 re[2][2], im[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) re[i][j] = im[i][j] = doublex4{0.0, 0.0, 0.0, 0.0};
  // element q = tid + 256 j of a 16 x 64 stage: sample q / 64, column q % 64
  const bool ra_ok = r0 + (tid & 63) < a.K, rb_ok = c0 + (tid & 63) < a.K;
  double2 va[4], vb[4];
  auto gload = [&](int64_t n) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t nn = n + (tid >> 6) + 4 * j;
      const double2* row = a.X + nn * a.K + (tid & 63);
      va[j] = vb[j] = make_double2(0.0, 0.0);
      if (nn < n1 && ra_ok) va[j] = row[r0];
      if (nn < n1 && rb_ok) vb[j] = row[c0];
    }
  };
  auto sstore = [&](int buf) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      As[buf][(tid >> 6) + 4 * j][tid & 63] = va[j];
      Bs[buf][(tid >> 6) + 4 * j][tid & 63] = vb[j];
    }
  };
  if (n0 < n1) {
    gload(n0);
    sstore(0);
  }
  __syncthreads();
  int buf = 0;
  for (int64_t n = n0; n < n1; n += HS) {
    const bool more = n + HS < n1;
    if (more) gload(n + HS);
#pragma unroll
    for (int ks = 0; ks < HS / 4; ++ks) {
      double2 fa[2], fb[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        fa[i] = As[buf][ks * 4 + lk][wr * 32 + i * 16 + li];
        fb[i] = Bs[buf][ks * 4 + lk][wc * 32 + i * 16 + li];
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          re[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[i].x, fb[j].x, re[i][j], 0, 0, 0);
          if (!REAL) im[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[i].x, fb[j].y, im[i][j], 0, 0, 0);
        }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          re[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[i].y, fb[j].y, re[i][j], 0, 0, 0);
          if (!REAL) im[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(-fa[i].y, fb[j].x, im[i][j], 0, 0, 0);
        }
    }
    if (more) sstore(buf ^ 1);  // the other buffer: its readers passed the last barrier
    __syncthreads();
    buf ^= 1;
  }
  double* part = a.part ? a.part + ((size_t)blockIdx.y * a.ntiles + blockIdx.x) * (REAL ? 1 : 2) * HT * HT : nullptr;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = wr * 32 + i * 16 + lk + 4 * r, col = wc * 32 + j * 16 + li;
        const double2 v = make_double2(re[i][j][r], REAL ? 0.0 : im[i][j][r]);
        if (!part)
          h64_put(a, r0 + row, c0 + col, v);
        else if (REAL)
          part[row * HT + col] = v.x;
        else
          ((double2*)part)[row * HT + col] = v;
      }
}

// S from the nsplit partial tiles, added in order
template <bool REAL>
__global__ __launch_bounds__(256) void k_herk64_add(h64_args a, int nsplit) {
  int tr, tc;
  h64_tile(blockIdx.x, tr, tc);
  const int e = blockIdx.y * 256 + threadIdx.x;
  double2 v = make_double2(0.0, 0.0);
  for (int z = 0; z < nsplit; ++z) {
    const size_t at = ((size_t)z * a.ntiles + blockIdx.x) * HT * HT + e;
    if (REAL)
      v.x += a.part[at];
    else
      v = cadd(v, ((const double2*)a.part)[at]);
  }
  h64_put(a, (int64_t)tr * HT + e / HT, (int64_t)tc * HT + e % HT, v);
}

int64_t h64_tiles(int64_t K) {
  const int64_t t = (K + HT - 1) / HT;
  return t * (t + 1) / 2;
}

size_t split_bytes(int64_t K, bool real) { return sizeof(double) * (real ? 1 : 2) * HT * HT * (size_t)h64_tiles(K); }

}  // namespace

// Sample ranges: two rounds of resident groups (two a compute unit) at 64 samples a range
// or more, where the tiles alone do not fill the chip; as many as `room` bytes of scratch hold.
int herk64_splits(int64_t N, int64_t K, int mode, size_t room) {
  const int64_t want = std::min<int64_t>(1024 / h64_tiles(K), N / 64);
  const int64_t fit = (int64_t)(room / split_bytes(K, mode == VMC_SR_REAL));
  return (int)std::max<int64_t>(1, std::min(want, fit));
}

size_t herk64_ws_bytes(int64_t K, int mode, int nsplit) {
  return nsplit > 1 ? split_bytes(K, mode == VMC_SR_REAL) * nsplit : 0;
}

void herk_f64(vmc_ctx* ctx, const double2* X, int64_t N, int64_t K, int mode, double nu, double eps,
              double2* S, double2* diag, void* ws, int nsplit) {
  h64_args a{};
  a.X = X;
  a.N = N;
  a.K = K;
  a.per = ((N + nsplit - 1) / nsplit + HS - 1) / HS * HS;
  a.mode = mode;
  a.nu = nu;
  a.eps = eps;
  a.S = S;
  a.diag = diag;
  a.part = nsplit > 1 ? (double*)ws : nullptr;
  a.ntiles = (int)h64_tiles(K);
  const dim3 grid((unsigned)a.ntiles, (unsigned)nsplit);
  const dim3 grid2((unsigned)a.ntiles, HT * HT / 256);
  if (mode == VMC_SR_REAL) {
    k_herk64<true><<<grid, 256, 0, ctx->stream>>>(a);
    if (nsplit > 1) k_herk64_add<true><<<grid2, 256, 0, ctx->stream>>>(a, nsplit);
  } else {
    k_herk64<false><<<grid, 256, 0, ctx->stream>>>(a);
    if (nsplit > 1) k_herk64_add<false><<<grid2, 256, 0, ctx->stream>>>(a, nsplit);
  }
  VMC_HIP(hipGetLastError());
}
