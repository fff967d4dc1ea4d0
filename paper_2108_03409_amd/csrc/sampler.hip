// Metropolis sampler (Sec. 2.1 and Sec. 4.2 "Sampler"): all chains advance in
// sync, one or two wavefronts per chain, the chain's hidden units spread over
// the lanes (t_j = tanh theta_j in registers).  A proposal costs N_h/64 complex
// multiply-adds per lane plus one wave reduction, using the move identity of
// rbm.hip:
//   2 Re(log psi(s') - log psi(s)) = 2 Re(-2 sigma_m alpha_m + LC_m)
//                                    + sum_j log|1 - sigma_m t_j T_jm|^2.
// On acceptance t_j follows the tanh addition rule
// t' = (t - sigma T) / (1 - sigma t T).  With flips and exchanges theta is formed from
// the spins at the start of a call and then follows the accepted moves in registers to its
// end; every record forms t and log psi anew from it.
//
// VMC_PROP_MADE_MIX: each sweep starts with global Metropolis-Hastings steps
// made by all chains together (mixsampler.hip; the proposals of the next step
// are formed on a second stream during the sweep); the sweep's single-spin
// flips then run here, one launch per sweep, and the matrix cores form each
// chain's theta for the next global step and the record from its spins.
#include "internal.h"

using namespace dev;

namespace {

struct sampler_args {
  const double2* params;
  const double2* Wt;
  const double2* D;  // [n_moves][N_h]
  const double2* T;  // [n_moves][N_h]
  const double2* LC;
  const double2* alpha;
  const int2* bonds;
  int n_moves;
  int proposal;  // VMC_PROP_FLIP / VMC_PROP_EXCHANGE / VMC_PROP_MADE_MIX
  int N, W, Nh;
  int n_chains;
  uint64_t* bits;
  uint2 key;
  uint64_t t0;
  int init;             // draw initial states
  int64_t therm_steps;  // proposals before the first record
  int64_t n_record;
  int sweep;
  uint64_t* s_out;
  double2* logpsi_out;
  unsigned long long* acc;  // [n_chains] accepted proposals (added to)
  const double2* theta;     // [n_chains][N_h] theta of the chains' spins (NULL: rebuilt here)
};

// One chain per work-group of NW waves.  With NW = 2 wave w takes the hidden
// units j = 64 Q w + 64 q + lane; both waves keep their own copy of the
// configuration and of the step tables and reach the same decisions, exchanging
// only their partial ratio (mantissa and exponent) through LDS behind one
// barrier per proposal.  The configuration and the draws of 64 steps lie over the
// lanes, and everything a proposal takes from them (its move, site, spin and the
// ratio it needs) is read by lane number into scalar registers, so that the chain's
// dependent path holds no LDS read and the rows are addressed without vector
// arithmetic.  TRACK: theta follows the accepted moves, and every record forms log
// psi and t anew from it; without it (global proposals) the caller does so between
// launches, and the row of D is not read at all.
// Bound: the dependent path of ratio, reduction, decision and update at one or two
// waves per SIMD; with many chains the vector instructions and the row of T (12.8 KB
// a proposal at N_h = 800) from L2.  Waves per SIMD: without TRACK three where the
// registers allow (20 x 20: 11.1 ms for 4 sweeps instead of 12.1 with two; seven slots spill
// 8 to 11 registers with and without TRACK); the
// two-wave groups of few chains are held to two, without which the dispatcher
// leaves three on some SIMDs and one on others (Heisenberg 10 x 10: 0.92 instead of 0.79 ms).
// Eight slots with TRACK have one wave per SIMD, whose 512 registers hold them: held to two
// they kept 84 of theirs in scratch memory (64 sites, flips, 512 units, 4 096 chains x 2
// sweeps 1.10 instead of 0.64 ms; 1 024 units, 1 024 chains, one sweep 0.40 instead of 0.23).
// 20 x 20, N_h = 800, 4 096 chains: 8.25 -> 1.8 ms a sweep; Heisenberg 10 x 10,
// N_h = 400, 1 024 chains x 8 sweeps 1.13 -> 0.75 ms, 4 096 chains x 4 sweeps
// 2.36 -> 1.0 ms (theta in LDS, rows of T and D per proposal, step tables in LDS,
// one wave of 16 slots per chain above 512 units before).
template <int Q, int NW, bool TRACK>
__global__ __launch_bounds__(64 * NW)
__attribute__((amdgpu_waves_per_eu(TRACK && Q > 7 ? 1 : TRACK || Q > 7 || (NW == 2 && Q <= 4) ? 2 : 3,
                                   NW == 2 && (TRACK || Q <= 4) ? 2 : 8))) void k_metropolis(sampler_args a) {
  __shared__ uint64_t cbs[NW][64];  // chain configuration, W <= 64 words (one copy per wave)
  __shared__ double pm_s[2][NW];  // partial ratios of the waves, alternating over the exchanges
  __shared__ int pe_s[2][NW];
  __shared__ double2 lp_s[NW];
  const int c = blockIdx.x;
  if (c >= a.n_chains) return;
  const int lane = threadIdx.x & 63;
  const int wv = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  uint64_t* cb = cbs[wv];
  const int jb = 64 * Q * wv;  // first hidden unit of this wave
  const int N = a.N, W = a.W, Nh = a.Nh;

  if (a.init) {
    if (lane == 0) {
      if (a.proposal != VMC_PROP_EXCHANGE) {
        for (int w = 0; w < W; ++w) {
          uint4 y = philox(make_uint4((uint32_t)c, (uint32_t)(w >> 1), 0u, 2u), a.key);
          uint64_t word = (w & 1) ? ((uint64_t)y.z | ((uint64_t)y.w << 32)) : ((uint64_t)y.x | ((uint64_t)y.y << 32));
          const int rem = N - 64 * w;
          if (rem < 64) word &= (1ull << rem) - 1ull;
          cb[w] = word;
        }
      } else {
        for (int w = 0; w < W; ++w) cb[w] = 0ull;
        for (int i = 0; i < N / 2; ++i) cb[i >> 6] |= 1ull << (i & 63);
        for (int i = N - 1; i >= 1; --i) {
          uint4 y = philox(make_uint4((uint32_t)c, (uint32_t)i, 1u, 2u), a.key);
          const int j = (int)to_index(y.x, (uint32_t)(i + 1));
          const uint64_t bi = (cb[i >> 6] >> (i & 63)) & 1ull, bj = (cb[j >> 6] >> (j & 63)) & 1ull;
          if (bi != bj) {
            cb[i >> 6] ^= 1ull << (i & 63);
            cb[j >> 6] ^= 1ull << (j & 63);
          }
        }
      }
    }
  } else {
    for (int w = lane; w < W; w += 64) cb[w] = a.bits[(int64_t)c * W + w];
  }
  __syncthreads();

  // theta_j = b_j + sum_i W_ji sigma_i for the lane's hidden units, four sites'
  // rows in flight; 0 past N_h
  double2 tt[Q], th[Q];
  auto build_theta = [&] {
    int64_t at[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int j = jb + lane + 64 * q;
      at[q] = j < Nh ? j : Nh - 1;
      th[q] = a.params[N + at[q]];
    }
#pragma unroll 4
    for (int i = 0; i < N; ++i) {
      const double sg = ((cb[i >> 6] >> (i & 63)) & 1ull) ? 1.0 : -1.0;
      const double2* w = a.Wt + (int64_t)i * Nh;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const double2 v = w[at[q]];
        th[q] = make_double2(fma(sg, v.x, th[q].x), fma(sg, v.y, th[q].y));
      }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (jb + lane + 64 * q >= Nh) th[q] = make_double2(0.0, 0.0);
  };
  if (a.theta) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int j = jb + lane + 64 * q;
      th[q] = j < Nh ? a.theta[(int64_t)c * Nh + j] : make_double2(0.0, 0.0);
    }
  } else {
    build_theta();
  }
  // t = tanh theta, and the sum of log cosh theta over the lane's units:
  // one unit at a time through lane-private LDS slots, so that the elementary functions
  // stand in the code once and the loop over the proposals stays in the instruction cache
  __shared__ double2 ths[NW][Q][64];
  auto tanh_theta = [&] {
    double2 lp = make_double2(0.0, 0.0);
#pragma unroll
    for (int q = 0; q < Q; ++q) ths[wv][q][lane] = th[q];
#pragma unroll 1
    for (int q = 0; q < Q; ++q) {
      double2 t, l;
      ctanh_logcosh(ths[wv][q][lane], t, l);
      if (jb + lane + 64 * q < Nh) lp = cadd(lp, l);
      ths[wv][q][lane] = t;
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) tt[q] = ths[wv][q][lane];
    return lp;
  };
  tanh_theta();

  unsigned long long accepted = 0;
  const int64_t total = a.therm_steps + a.n_record * a.sweep;
  // The move of step t + 1 is known from its counter before step t resolves:
  // its row of T is loaded one step ahead.
  // The counters of 64 consecutive steps are drawn together, one per lane, into
  // a table of moves and of the ratio each needs to be accepted (the same Philox
  // values as one per step).  accept iff L = sum_j log |f_j|^2 > log u - c,
  // c = 2 Re(-2 sigma alpha + LC), without a logarithm on the chain's path: each
  // lane's product of |f|^2 as mantissa in [1/2, 1) and exponent, the wave's
  // product M 2^E (M >= 2^-64, no underflow), and M 2^E > e^(log u - c) tested as
  // ldexp(M, E - n) > 2^r with (log u - c) / ln 2 = n + r, n integer, r in [0, 1):
  // n and 2^r of both values of sigma stand in the table.  Decides as
  // log u < c + L except within rounding of a tie.  Step s of a group of 64 stands
  // in lane s of its registers.
  struct draw_t {
    int m, x;        // move; its sites (first | second << 16)
    double p2[2];    // [sigma > 0]
    int n2[2];
  };
  // entries of the lane's units in row m of a [n_moves][N_h] table, zero past N_h
  // (out of the buffer's range, which the hardware checks as lane offset against range -
  // scalar offset, 1024 q being below the range: a unit past N_h has t = 0 and T = 0, hence
  // f = 1 and no change)
  auto load_row = [&](const double2* tab, int m, double2(&r)[Q]) {
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(tab + (int64_t)m * Nh), 0, Nh * 16, 0x00027000);
#pragma unroll
    for (int q = 0; q < Q; ++q)
      r[q] = __builtin_bit_cast(double2,
                                __builtin_amdgcn_raw_buffer_load_b128(rsrc, (jb + lane) * 16, 1024 * q, 0));
  };
  const int exch = a.proposal == VMC_PROP_EXCHANGE;
  auto draw64 = [&](int64_t s0) {
    const uint64_t tl = a.t0 + (uint64_t)(s0 + lane);
    const uint4 y = philox(make_uint4((uint32_t)c, (uint32_t)tl, (uint32_t)(tl >> 32), 0u), a.key);
    draw_t d;
    d.m = d.x = (int)to_index(y.x, (uint32_t)a.n_moves);
    const double lu = log(to_uniform(y.y, y.z));
    const double2 al = a.alpha[d.m], lc = a.LC[d.m];
    if (exch) {
      const int2 bd = a.bonds[d.m];
      d.x = bd.x | (bd.y << 16);
    }
#pragma unroll
    for (int up = 0; up < 2; ++up) {
      const double sg = up ? 1.0 : -1.0;
      const double t2 =
          fmin(fmax((lu - 2.0 * (-2.0 * sg * al.x + lc.x)) * 1.4426950408889634074, -4096.0), 4096.0);
      const double n2 = floor(t2);
      d.p2[up] = exp2(t2 - n2);
      d.n2[up] = (int)n2;
    }
    return d;
  };
  auto rl = [](int v, int i) { return __builtin_amdgcn_readlane(v, i); };
  // the configuration, word w in lane w
  uint32_t cl = lane < W ? (uint32_t)cb[lane] : 0u, ch = lane < W ? (uint32_t)(cb[lane] >> 32) : 0u;
  auto spin_up = [&](int i) {
    const uint32_t w = i & 32 ? (uint32_t)__builtin_amdgcn_readlane((int)ch, i >> 6)
                              : (uint32_t)__builtin_amdgcn_readlane((int)cl, i >> 6);
    return (w >> (i & 31)) & 1u;
  };
  auto flip = [&](int i) {
    const uint32_t b = lane == (i >> 6) ? 1u << (i & 31) : 0u;
    cl ^= i & 32 ? 0u : b;
    ch ^= i & 32 ? b : 0u;
  };
  // Two sets of row registers alternate between the current step and the next
  // (the loop runs two steps per trip), so that no row is copied from one set to
  // the other; rows two and three steps ahead measured no faster.
  double2 TR[2][Q];
  int mr[2], xr[2];
  // TRACK: theta, and the row of D the last accepted move adds to it (factor dsg,
  // zero after a rejection, when the row asked for is the first one, a hit in L1)
  constexpr int QT = TRACK ? Q : 1;
  double2 DP[QT];
  double dsg = 0.0;
#pragma unroll
  for (int q = 0; q < QT; ++q) DP[q] = make_double2(0.0, 0.0);
  int par = 0;  // buffer of the waves' exchange, alternating over the exchanges
  draw_t cur = draw64(0);
  mr[0] = rl(cur.m, 0);
  xr[0] = rl(cur.x, 0);
  load_row(a.T, mr[0], TR[0]);
  int64_t to_record = a.therm_steps + a.sweep, row = c;  // steps to the next record, its row
  for (int64_t s0 = 0; s0 < total; s0 += 2) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int64_t step = s0 + h;
    if (h > 0 && step >= total) break;
    const int i = (int)(step & 63);
    const double2(&Tc)[Q] = TR[h];
    const int m = mr[h], x = xr[h];
    const int site = exch ? x & 0xffff : x, site2 = x >> 16;
    const uint32_t up = spin_up(site);
    const double p2 = up ? readlane_f64(cur.p2[1], i) : readlane_f64(cur.p2[0], i);
    const int n2 = up ? rl(cur.n2[1], i) : rl(cur.n2[0], i);
    if (h == 1 && i == 63 && step + 1 < total) cur = draw64(step + 1);
    mr[h ^ 1] = rl(cur.m, (i + 1) & 63);
    xr[h ^ 1] = rl(cur.x, (i + 1) & 63);
    load_row(a.T, mr[h ^ 1], TR[h ^ 1]);
    if (exch && up == spin_up(site2)) {
      ++accepted;  // the exchange changes nothing
    } else {
      const double sg = up ? 1.0 : -1.0;
      double prod = 1.0;
      // per hidden unit the factor f = 1 - sigma t_j T_jm and |f|^2
      double2 f[Q];
      double n[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const double2 p = cmul(tt[q], Tc[q]);
        f[q] = make_double2(1.0 - sg * p.x, -sg * p.y);
        n[q] = f[q].x * f[q].x + f[q].y * f[q].y;
        prod *= n[q];
      }
      int ex;
      const double mt = frexp(prod, &ex);
      double M = wave_prod_uniform(mt);
      int E = wave_isum_uniform(ex);
      if constexpr (NW > 1) {  // the other waves' units: every wave forms the same product
        if (lane == 0) {
          pm_s[par][wv] = M;
          pe_s[par][wv] = E;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        M = pm_s[par][0];
        E = pe_s[par][0];
#pragma unroll
        for (int w = 1; w < NW; ++w) {
          M *= pm_s[par][w];
          E += pe_s[par][w];
        }
        par ^= 1;
      }
      // one value for the work-group: a uniform decision
      const bool acc = __builtin_amdgcn_readfirstlane(ldexp(M, E - n2) > p2);
      if constexpr (TRACK) {
#pragma unroll
        for (int q = 0; q < Q; ++q)
          th[q] = make_double2(fma(-dsg, DP[q].x, th[q].x), fma(-dsg, DP[q].y, th[q].y));
        dsg = acc ? 2.0 * sg : 0.0;
        load_row(a.D, acc ? m : 0, DP);
      }
      if (acc) {
        ++accepted;
        // t' = (t - sigma T) / f = (t - sigma T) conj(f) / |f|^2, with 1 / |f|^2 from the
        // hardware reciprocal and two Newton steps (a zero factor gives a zero ratio, which
        // is never accepted)
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const double2 nu = make_double2(tt[q].x - sg * Tc[q].x, tt[q].y - sg * Tc[q].y);
          double inv = __builtin_amdgcn_rcp(n[q]);
          inv = fma(inv, fma(-n[q], inv, 1.0), inv);
          inv = fma(inv, fma(-n[q], inv, 1.0), inv);
          tt[q] = make_double2((nu.x * f[q].x + nu.y * f[q].y) * inv, (nu.y * f[q].x - nu.x * f[q].y) * inv);
        }
        flip(site);
        if (exch) flip(site2);
      }
    }
    // record after every completed sweep of the recording phase
    if (--to_record == 0) {
      to_record = a.sweep;
      if (wv == 0)
        if (lane < W) a.s_out[row * W + lane] = (uint64_t)cl | ((uint64_t)ch << 32);
      if constexpr (TRACK) {
#pragma unroll
        for (int q = 0; q < Q; ++q)
          th[q] = make_double2(fma(-dsg, DP[q].x, th[q].x), fma(-dsg, DP[q].y, th[q].y));
        dsg = 0.0;
        double2 lp = tanh_theta();
        if (wv == 0)
          for (int i = lane; i - lane < N; i += 64) {  // word i / 64 is the same in all lanes
            const uint32_t lo = (uint32_t)rl((int)cl, (i - lane) >> 6);
            const uint32_t hi = (uint32_t)rl((int)ch, (i - lane) >> 6);
            const uint32_t b = ((lane & 32 ? hi : lo) >> (lane & 31)) & 1u;
            if (i < N) lp = cadd(lp, cscale(a.params[i], b ? 1.0 : -1.0));
          }
        lp = wave_sum(lp);
        if constexpr (NW > 1) {  // records are rare: plain barriers around the exchange
          if (lane == 0) lp_s[wv] = lp;
          __syncthreads();
          lp = lp_s[0];
#pragma unroll
          for (int w = 1; w < NW; ++w) lp = cadd(lp, lp_s[w]);
          __syncthreads();
        }
        if (wv == 0 && lane == 0 && a.logpsi_out) a.logpsi_out[row] = lp;
      }
      row += a.n_chains;
    }
  }
  }
  if (wv == 0)
    if (lane < W) a.bits[(int64_t)c * W + lane] = (uint64_t)cl | ((uint64_t)ch << 32);
  if (wv == 0 && lane == 0) a.acc[c] += accepted;
}

__global__ void k_zero_u64(unsigned long long* p, int64_t n) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e < n) p[e] = 0ull;
}

// Two waves per chain above 512 hidden units (eight slots of 64 fill one wave's
// registers), and above 128 when the chains leave SIMDs idle (at most one chain
// per SIMD).  1 024 chains: Heisenberg 10 x 10, N_h = 400, 8 sweeps 0.79 ms with
// two waves, 0.90 with one, 0.91 with four; flips 8 x 8, N_h = 256, 16 sweeps 0.93,
// 1.10, 1.17; one slot per lane (N_h = 20, 512 chains) 0.30 with two, 0.22 with one.
// 4 096 chains: N_h = 400 2.07 with two, 1.0 with one; N_h = 256 0.76, 0.55.
template <bool TRACK>
void launch(vmc_ctx* ctx, const sampler_args& a, hipStream_t st) {
  const int nw = a.Nh > 512 || (a.Nh > 128 && a.n_chains <= 4 * cu_count(ctx)) ? 2 : 1;
  const int q = (a.Nh + 64 * nw - 1) / (64 * nw);
  const dim3 grid(a.n_chains), blk(64 * nw);
  switch (nw * 16 + q) {
#define CASE(Q, NW) \
  case NW * 16 + Q: k_metropolis<Q, NW, TRACK><<<grid, blk, 0, st>>>(a); break
    CASE(1, 1);
    CASE(2, 1);
    CASE(3, 1);
    CASE(4, 1);
    CASE(5, 1);
    CASE(6, 1);
    CASE(7, 1);
    CASE(8, 1);
    CASE(2, 2);
    CASE(3, 2);
    CASE(4, 2);
    CASE(5, 2);
    CASE(6, 2);
    CASE(7, 2);
    CASE(8, 2);
#undef CASE
    default: throw vmc_error{VMC_ERR_UNSUPPORTED, "sampler supports up to 1024 hidden units"};
  }
  VMC_HIP(hipGetLastError());
}

// [nc][Nh] theta for the duration of a call, from the context's workspace: up to 1 GiB (what
// log psi of 65 536 configurations of 1 024 units takes) and within its limit; otherwise
// NULL, and the kernel forms theta itself
double2* scratch_theta(vmc_ctx* ctx, int64_t nc, int Nh) {
  const size_t bytes = ws_round(sizeof(double2) * (size_t)nc * Nh);
  if (bytes > (size_t)1 << 30 || (ctx->ws_limit && bytes > ctx->ws_limit)) return nullptr;
  try {
    ws_reserve(ctx, bytes);
  } catch (const vmc_error& e) {
    if (e.code != VMC_ERR_OOM) throw;
    return nullptr;
  }
  return (double2*)ws_take(ctx, bytes);
}

}  // namespace

void sampler_run(vmc_sampler* S, int64_t n_per_chain, uint64_t* s_out, double2* logpsi_out) {
  vmc_model* m = S->model;
  VMC_REQUIRE(m->kind == MODEL_RBM, "sampler supports RBM models");
  VMC_REQUIRE(m->W <= 64, "sampler supports up to 4096 sites");
  const int move_kind = S->opts.proposal == VMC_PROP_EXCHANGE ? 1 : 0;
  rbm_ensure_tables(m, S->ham, move_kind);
  const rbm_move_tables& tb = m->tab[move_kind];
  const int nc = S->opts.n_chains;
  hipStream_t st = S->ctx->stream;
  sampler_args a{};
  a.params = m->params;
  a.Wt = m->Wt;
  a.T = tb.Tt;
  a.D = tb.Dt;
  a.LC = tb.LC;
  a.alpha = tb.alpha;
  a.bonds = S->ham->bonds;
  a.n_moves = tb.n_moves;
  a.proposal = S->opts.proposal;
  a.N = m->N;
  a.W = m->W;
  a.Nh = m->Nh;
  a.n_chains = nc;
  a.bits = S->bits;
  a.key = make_uint2((uint32_t)S->opts.seed, (uint32_t)(S->opts.seed >> 32));
  a.acc = S->acc;
  a.sweep = S->opts.sweep_steps;
  k_zero_u64<<<grid_for(3 * (int64_t)nc, 256), 256, 0, st>>>(S->acc, 3 * (int64_t)nc);
  if (S->opts.proposal != VMC_PROP_MADE_MIX) {
    a.t0 = S->t;
    a.init = !S->bits_valid;
    a.therm_steps = S->thermalized ? 0 : (int64_t)S->opts.therm_sweeps * S->opts.sweep_steps;
    a.n_record = n_per_chain;
    a.s_out = s_out;
    a.logpsi_out = logpsi_out;
    // theta of the chains' spins by the matrix cores where the kernel's own serial sum over
    // the sites costs more than a launch (a call of 16 proposals, 1 024 chains: 100 sites, 400
    // units 79 against 66 us; 64 sites, 256 units 55 against 54; 48 sites, 192 units equal; 64
    // chains of 64 sites and units 38 against 41); the first call draws its spins in the
    // kernel and keeps that sum
    if (!a.init && m->N >= 48) {
      if (double2* theta = scratch_theta(S->ctx, nc, m->Nh)) {
        rbm_theta(m, S->bits, nc, theta);
        a.theta = theta;
      }
    }
    launch<true>(S->ctx, a, st);
    S->t += (uint64_t)(a.therm_steps + a.n_record * a.sweep);
    S->thermalized = 1;
    S->bits_valid = 1;
    return;
  }
  // MADE_MIX: per sweep, global_steps global steps of all chains, then one
  // launch of the sweep's flips; the chains' theta (S->mix_theta) is formed on the
  // matrix cores from their spins after every launch
  mix_ensure(S);
  a.t0 = S->t;
  a.init = !S->bits_valid;
  a.therm_steps = 0;
  a.n_record = 0;
  if (a.init) launch<false>(S->ctx, a, st);  // initial states (first call), no proposals
  rbm_theta(m, S->bits, nc, S->mix_theta);
  S->bits_valid = 1;
  a.init = 0;
  a.theta = S->mix_theta;
  const int64_t n_therm = S->thermalized ? 0 : S->opts.therm_sweeps;
  for (int64_t sw = 0; sw < n_therm + n_per_chain; ++sw) {
    for (int gs = 0; gs < S->opts.global_steps; ++gs) mix_global_step(S, S->g++);
    const bool rec = sw >= n_therm;
    a.t0 = S->t;
    a.therm_steps = rec ? 0 : a.sweep;
    a.n_record = rec ? 1 : 0;
    a.s_out = rec ? s_out + (sw - n_therm) * (int64_t)nc * m->W : nullptr;
    launch<false>(S->ctx, a, st);
    S->t += (uint64_t)a.sweep;
    rbm_theta(m, S->bits, nc, S->mix_theta);
    if (rec && logpsi_out) rbm_log_psi_theta(m, S->bits, nc, S->mix_theta, logpsi_out + (sw - n_therm) * (int64_t)nc);
  }
  mix_wait_side(S);
  S->thermalized = 1;
}

namespace {
__global__ void k_copy_made(const double* __restrict__ W1mT, const double* __restrict__ W2m,
                            const double* __restrict__ params, int N, int H, double* __restrict__ buf) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t nh = (int64_t)N * H;
  if (e < nh) {
    buf[e] = W1mT[e];
    buf[nh + e] = W2m[e];
  }
  if (e < H) buf[2 * nh + e] = params[nh + e];
  if (e < N) buf[2 * nh + H + e] = params[2 * nh + H + e];
}
}  // namespace

// work buffers of the global steps (allocated on first use)
void mix_ensure(vmc_sampler* S) {
  const int64_t nc = S->opts.n_chains;
  if (!S->mix_tf) {  // the teacher-forcing workspace depends on the proposal's hidden size
    VMC_HIP(hipMalloc(&S->mix_tf, sizeof(double) * nc * ((int64_t)S->N + S->made_H)));
  }
  if (S->mix_prop) return;
  VMC_HIP(hipMalloc(&S->mix_prop, sizeof(uint64_t) * 2 * nc * S->W));
  VMC_HIP(hipMalloc(&S->mix_lq, sizeof(double) * 3 * nc));
  VMC_HIP(hipMalloc(&S->mix_theta, sizeof(double2) * nc * S->model->Nh));
  VMC_HIP(hipMalloc(&S->mix_theta_prop, sizeof(double2) * 2 * nc * S->model->Nh));
  VMC_HIP(hipStreamCreateWithFlags(&S->mix_side, hipStreamNonBlocking));
  VMC_HIP(hipEventCreateWithFlags(&S->mix_ev_main, hipEventDisableTiming));
  for (auto& e : S->mix_ev_prop) VMC_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
}

void mix_release(vmc_sampler* S) {
  if (S->mix_side) (void)hipStreamSynchronize(S->mix_side);
  for (void* p : {(void*)S->mix_prop, (void*)S->mix_lq, (void*)S->mix_theta, (void*)S->mix_theta_prop, (void*)S->mix_tf})
    if (p) (void)hipFree(p);
  S->mix_prop = nullptr;
  S->mix_lq = nullptr;
  S->mix_theta = S->mix_theta_prop = nullptr;
  S->mix_tf = nullptr;
  for (auto& e : S->mix_ev_prop)
    if (e) (void)hipEventDestroy(e);
  if (S->mix_ev_main) (void)hipEventDestroy(S->mix_ev_main);
  if (S->mix_side) (void)hipStreamDestroy(S->mix_side);
  S->mix_ev_prop[0] = S->mix_ev_prop[1] = S->mix_ev_main = nullptr;
  S->mix_side = nullptr;
  S->mix_pg[0] = S->mix_pg[1] = ~0ull;
}

extern "C" int vmc_sampler_set_proposal_made(vmc_sampler* S, const vmc_made* md) {
  if (!S || !md) return VMC_ERR_INVALID_ARG;
  try {
    VMC_REQUIRE(md->ctx == S->ctx, "MADE belongs to another context");
    VMC_REQUIRE(md->N == S->N, "MADE input size differs from the sampler's site count");
    VMC_REQUIRE(md->H <= 1024, "MADE hidden size above 1024");
    VMC_HIP(hipSetDevice(S->ctx->device));
    VMC_REQUIRE(mix_made_fits(md->H, md->W),
                "MADE proposal too large for the batched global step (its pre-activations for 16 chains must fit "
                "in one work-group's LDS)");
    const int64_t nh = (int64_t)md->N * md->H;
    const size_t bytes = sizeof(double) * (size_t)(2 * nh + md->H + md->N);
    std::vector<int> perm, mstart;
    mix_made_layout(md->N, md->H, perm, mstart);
    perm.insert(perm.end(), mstart.begin(), mstart.end());
    VMC_HIP(hipStreamSynchronize(S->ctx->stream));
    if (S->mix_side) VMC_HIP(hipStreamSynchronize(S->mix_side));
    S->mix_pg[0] = S->mix_pg[1] = ~0ull;  // proposals of the previous network
    if (S->mix_tf) VMC_HIP(hipFree(S->mix_tf));
    S->mix_tf = nullptr;
    if (S->made_buf) VMC_HIP(hipFree(S->made_buf));
    if (S->mix_perm) VMC_HIP(hipFree(S->mix_perm));
    S->made_buf = nullptr;
    S->mix_perm = nullptr;
    S->made_H = 0;
    VMC_HIP(hipMalloc(&S->made_buf, bytes));
    VMC_HIP(hipMalloc(&S->mix_perm, sizeof(int) * perm.size()));
    VMC_HIP(hipMemcpy(S->mix_perm, perm.data(), sizeof(int) * perm.size(), hipMemcpyHostToDevice));
    S->made_H = md->H;
    const int64_t n = std::max<int64_t>(nh, std::max(md->H, md->N));
    k_copy_made<<<grid_for(n, 256), 256, 0, S->ctx->stream>>>(md->W1mT, md->W2m, md->params, md->N, md->H,
                                                               S->made_buf);
    VMC_HIP(hipGetLastError());
    S->ctx->err.clear();
    return VMC_OK;
  } catch (vmc_error& e) {
    S->ctx->err = e.msg;
    return e.code;
  }
}
