// Vectorised stock-trading environment: observation assembly, Gaussian action
// sampling, trade execution, reward, episode end and reset (Table 1 and
// Sec. 5.3 of the paper; the worker of Sec. 4.2 steps N such envs at once),
// plus the per-env state plumbing and the leaderboard reduction (Sec. 4.1).
//
// This translation unit is compiled with floating-point contraction off: the
// share counts are decided by a fixed sequence of binary32 operations with one
// rounding each, and a fused multiply-add would change which integer a
// quotient lands on.
#include "pod_internal.h"

namespace pod {

namespace {

constexpr int kThreads = 256;

struct RowInfo {
  int32_t row_now;   // market row the trades execute at
  int32_t row_val;   // market row the portfolio is valued at (cursor + 1)
  int32_t row_obs;   // market row of the next observation (0 after a reset)
  int32_t done;
};

__device__ inline RowInfo rows_of(const EnvDims &d, int32_t tau, int32_t start, int32_t n) {
  const int32_t m = d.M == 1 ? 0 : n;
  RowInfo r;
  r.row_now = tau * d.M + m;
  r.row_val = (tau + 1) * d.M + m;
  r.done = (tau + 1 - start == d.H);
  r.row_obs = r.done ? start * d.M + m : r.row_val;
  return r;
}

// ------------------------------------------------------------------ observe
// obs[n] = [cash s0, price s1, holdings s2, indicators s3] at the current cursor; and its bf16 copy.
__global__ __launch_bounds__(kThreads) void observe_kernel(EnvDims d, EnvState s, const float *__restrict__ price,
                                                          const float *__restrict__ ind, float *__restrict__ obs,
                                                          ObsShadow sh) {
  // one wavefront per env row, lanes across the row
  const int lane = threadIdx.x & 63;
  const int n = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
  if (n >= d.N) return;
  const int32_t tau = s.tau[n];
  const int32_t m = d.M == 1 ? 0 : n;
  const size_t row = (size_t)tau * d.M + m;
  float *o = obs + (size_t)n * d.S;
  const int D = d.D, DK = D * d.K;
  __bf16 *sp = sh.p ? reinterpret_cast<__bf16 *>(sh.p) + (size_t)n * sh.pitch : nullptr;
#pragma unroll 4
  for (int j = lane; j < DK; j += 64) {
    const float v = ind[row * DK + j] * d.s_ind;
    o[1 + 2 * D + j] = v;
    if (sp) sp[j] = (__bf16)v;
  }
#pragma unroll 2
  for (int j = lane; j < D; j += 64) {
    const float p = price[row * D + j] * d.s_price, h = (float)s.h[(size_t)n * D + j] * d.s_hold;
    o[1 + j] = p;
    o[1 + D + j] = h;
    if (sp) sp[DK + 1 + j] = (__bf16)p, sp[DK + 1 + D + j] = (__bf16)h;
  }
  if (lane == 0) {
    const float c = s.cash[n] * d.s_cash;
    o[0] = c;
    if (sp) sp[DK] = (__bf16)c;
  }
  if (sp)
    for (int j = d.S + lane; j < sh.cols; j += 64) sp[j] = (__bf16)0.0f;
}

// ----------------------------------------------------------------- env step
// 512 threads step E envs: TPE = 512 / E neighbouring threads own one env, and a thread the stocks tl, tl + TPE, ...
// (at most ND) of its env, whose prices, holdings and orders stay in its registers from the first load to the last
// store.  What bounds the step is a chain: cursor -> prices -> orders -> the serial walk over the purchases -> holdings;
// everything else hangs off it:
//  - the cursor is read by every thread of an env (no barrier in front of the prices), the market part of the next
//    observation is requested together with the prices and written while the orders are packed;
//  - the ledger adds the sales from a dense row, and walks only the purchases: the threads pack them into a list in
//    stock order (ballots inside a wavefront, counts per 32 or 64 stocks across).  It runs in the env's own wavefront
//    (half) and needs one dependent operation per purchase while the cash lasts, none for a purchase it does not
//    buy a single share of, and the quotient only in between (13.5 -> 1.8 us of a step with 250 purchases);
//  - the account values before and after are sums over the env's threads in binary64.
// Measured per step: 2048 envs x 500 stocks x 4 indicators 106 -> 18.5 us, 5000 x 100 x 8 30 -> 15 us, 4096 x 30 x 8
// 11.2 -> 6.4 us, 16 x 5 x 2 6.0 -> 4.8 us (before: order slots of up to 32 envs and a ledger over all of them in LDS,
// holdings stored stock-major and hence moved in short runs).  The bytes of the first of these take 10 us.
constexpr int kEnvThreads = 512;
typedef float env_f32x4 __attribute__((ext_vector_type(4)));

struct __attribute__((aligned(16))) Purchase {
  float k, u;   // wanted shares, unit cost
  double rcp;   // 1 / u in binary64
};

__device__ inline double sum_lanes(double v, int width) {
  for (int o = 1; o < width; o *= 2) v += __shfl_xor(v, o);
  return v;
}

// s + v[0][0] + v[0][1] + ... in this order (two register sets, read one ahead of the other by hand, were slower)
__device__ inline float serial_sum(float s, const env_f32x4 *v, int n) {
#pragma unroll 8
  for (int c = 0; c < n; ++c) {
    const env_f32x4 x = v[c];
    s = s + x[0];
    s = s + x[1];
    s = s + x[2];
    s = s + x[3];
  }
  return s;
}

template <int E, int ND>
__global__ __launch_bounds__(kEnvThreads, 4) void env_step_kernel(EnvDims d, EnvState s, const float *__restrict__ price,
                                                                 const float *__restrict__ ind, StepIO io) {
  constexpr int TPE = kEnvThreads / E;        // threads per env
  constexpr int NI = ND == 1 ? 4 : 8;         // 16-byte indicator groups per thread that are requested with the prices
  constexpr int CW = TPE < 64 ? TPE : 64;               // stocks per count: the part of a wavefront one env has
  constexpr int NCW = TPE / CW, NC = ND * NCW;          // counts per pass over the stocks, per env
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const int D = d.D, DK = D * d.K, D4 = (D + 3) & ~3;
  const int lp = D | 1;                                      // (odd pitch in 16 bytes)
  Purchase *s_list = reinterpret_cast<Purchase *>(lds_raw);  // [E][lp] purchases in stock order
  float *s_sell = reinterpret_cast<float *>(s_list + E * lp);  // [E][D4] proceeds of the sales, 0 elsewhere
  const int sp_ = D4 + 4;
  float *s_sq = s_sell + E * sp_;                             // [E][sp_] squared noise
  const int op = D4 + 20;
  float *s_out = s_sq + E * sp_;                              // [E][op] outlay k u of the purchases, by list position
  int32_t *s_buy = reinterpret_cast<int32_t *>(s_out + E * op);  // [E][lp] shares bought, by list position
  double *s_part = reinterpret_cast<double *>(s_buy + E * lp + (E * lp & 1));  // [2][E][2] account value before / after
  float *s_e2 = reinterpret_cast<float *>(s_part + 4 * E);  // [E] sum of the squares
  int32_t *s_cnt = reinterpret_cast<int32_t *>(s_e2 + E);        // [E][NC]

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int e = tid / TPE, tl = tid & (TPE - 1), cw = tl / CW;  // cw: which wavefront of the env
  const int n0 = blockIdx.x * E, n = min(n0 + e, d.N - 1);
  const bool live = n0 + e < d.N;

  // -- requests that depend on nothing
  const int32_t tau = s.tau[n], start = s.start[n];
  const float cash_in = s.cash[n];
  float cash = cash_in, e2 = 0.0f;
  float mu[ND], eps[ND];
  int32_t h[ND];
  const size_t g0 = (size_t)n * D;
#pragma unroll
  for (int i = 0; i < ND; ++i) {
    const int dd = min(tl + TPE * i, D - 1);
    mu[i] = io.mu[g0 + dd];
    eps[i] = __builtin_nontemporal_load(io.noise + g0 + dd);
    h[i] = s.h[g0 + dd];
  }
  // -- and those that depend on the cursor
  const RowInfo ri = rows_of(d, tau, start, n);
  float pn[ND], pv[ND], po[ND];
#pragma unroll
  for (int i = 0; i < ND; ++i) {
    const int dd = min(tl + TPE * i, D - 1);
    pn[i] = price[(size_t)ri.row_now * D + dd];
    pv[i] = price[(size_t)ri.row_val * D + dd];
    po[i] = price[(size_t)ri.row_obs * D + dd];
  }
  const float *irow = ind + (size_t)ri.row_obs * DK;
  const int NG = DK / 4;  // whole groups of four indicators (rows need not be aligned)
  typedef env_f32x4 env_f32x4u __attribute__((aligned(4)));
  env_f32x4 iv[NI];
#pragma unroll
  for (int j = 0; j < NI; ++j) {
    const int g = tl + TPE * j;
    if (g < NG) iv[j] = *reinterpret_cast<const env_f32x4u *>(irow + 4 * g);
  }

  // -- orders
  float *o = io.obs_next + (size_t)n * d.S;
  __bf16 *sp = io.shadow.p ? reinterpret_cast<__bf16 *>(io.shadow.p) + (size_t)n * io.shadow.pitch : nullptr;
  int32_t q[ND], rank[ND];
  float unit[ND], kf[ND];
  double a0 = 0.0;
#pragma unroll
  for (int i = 0; i < ND; ++i) {
    const int dd = tl + TPE * i;
    const bool ok = live && dd < D;
    const float a_raw = mu[i] + d.sigma * eps[i];  // two roundings (contraction is off)
    const float ac = fminf(1.0f, fmaxf(-1.0f, a_raw));
    const int32_t k = ok ? (int32_t)truncf(ac * d.hmax) : 0;
    float sale = 0.0f;
    q[i] = 0;
    kf[i] = 0.0f;
    unit[i] = 0.0f;
    if (ok) {
      io.act_raw[g0 + dd] = a_raw;
      a0 += (double)h[i] * (double)pn[i];
    }
    if (k < 0) {
      const int32_t qs = min(-k, h[i]);
      h[i] -= qs;
      const float gross = pn[i] * (float)qs;
      sale = gross * d.one_minus_c;
      q[i] = -qs;
    } else if (k > 0) {
      kf[i] = (float)k;
      unit[i] = pn[i] * d.one_plus_c;
    }
    if (dd < D4) {
      s_sell[e * sp_ + dd] = sale;
      s_sq[e * sp_ + dd] = ok ? eps[i] * eps[i] : 0.0f;
    }
    const uint64_t all = __ballot(k > 0);
    const uint64_t mine = CW == 64 ? all : (all >> (lane & ~(CW - 1))) & ((1ull << (CW & 63)) - 1ull);
    const int cl = lane & (CW - 1);
    rank[i] = __popcll(mine & ((1ull << cl) - 1ull));
    if (cl == 0) s_cnt[e * NC + i * NCW + cw] = __popcll(mine);
  }
  a0 = sum_lanes(a0, CW);
  if ((lane & (CW - 1)) == 0) s_part[e * 2 + cw] = a0;
  __syncthreads();
  int total = 0;
  {
    int base[ND];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      if (NCW == 1 || c % NCW == 0) base[c / NCW] = total;
      if (NCW > 1 && c % NCW < cw) base[c / NCW] += s_cnt[e * NC + c];
      total += s_cnt[e * NC + c];
    }
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      rank[i] += base[i];
      if (kf[i] > 0.0f) {
        s_list[e * lp + rank[i]] = Purchase{kf[i], unit[i], 1.0 / (double)unit[i]};
        s_out[e * op + rank[i]] = kf[i] * unit[i];
      }
    }
    if (tl < 16) s_out[e * op + total + tl] = 0.0f;
  }
  // -- market part of the next observation
#pragma unroll
  for (int i = 0; i < ND; ++i) {
    const int dd = tl + TPE * i;
    if (live && dd < D) {
      const float v = po[i] * d.s_price;
      o[1 + dd] = v;
      if (sp) sp[DK + 1 + dd] = (__bf16)v;
    }
  }
  auto put = [&](int g, env_f32x4 v) {
    v[0] *= d.s_ind, v[1] *= d.s_ind, v[2] *= d.s_ind, v[3] *= d.s_ind;
    __builtin_nontemporal_store(v, reinterpret_cast<env_f32x4u *>(o + 1 + 2 * D + 4 * g));
    if (sp) {
      typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
      *reinterpret_cast<bf16x4 *>(sp + 4 * g) = bf16x4{(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
    }
  };
  if (live) {
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int g = tl + TPE * j;
      if (g < NG) put(g, iv[j]);
    }
  }
  __syncthreads();

  if (cw == NCW - 1 && io.logp) {
    // the squares in stock order (the log-probability is the same number in every schedule)
    const env_f32x4 *sq = reinterpret_cast<const env_f32x4 *>(s_sq + e * sp_);
    e2 = serial_sum(0.0f, sq, D4 / 4);
    if (NCW > 1 && (lane & (CW - 1)) == 0) s_e2[e] = e2;
  }
  if (cw == 0) {
    // -- the ledger (Table 1 actions: sell / buy / hold): all sales, then all purchases, in stock order, each limited
    // by the cash left:
    //   m = floor(cash / u); q = min(k, max(m, 0)); if (q u > cash) q -= 1; cash -= q u        (binary32)
    const env_f32x4 *sell = reinterpret_cast<const env_f32x4 *>(s_sell + e * sp_);
    cash = serial_sum(cash, sell, D4 / 4);
    const int cl = lane & (CW - 1);
    const Purchase *list = s_list + e * lp;
    auto affordable = [&](float c, float u) {  // of the CW entries the env's lanes hold: those the cash buys a share of
      const uint64_t all = __ballot(!(c < u));
      return CW == 64 ? all : (all >> (lane & ~(CW - 1))) & ((1ull << (CW & 63)) - 1ull);
    };
    for (int c0 = 0; c0 < total; c0 += CW) {
      const int p = c0 + cl;
      const Purchase mine = list[min(p, total - 1)];
      const float u = p < total ? mine.u : __builtin_inff();
      int32_t got = 0;
      for (int s0 = 0; s0 < CW && c0 + s0 < total; s0 += 16) {
        if (((affordable(cash, u) >> s0) & 0xffffull) == 0) continue;
        // sixteen purchases in full: as long as the balance stays clear of 0 (2^-20 of what it was, so every outlay
        // k u before it was below the balance by more than its own rounding), each quotient was at least k
        const env_f32x4 *out = reinterpret_cast<const env_f32x4 *>(s_out + e * op + c0 + s0);
        const float clear = cash * 0x1p-20f;
        float full = cash;
        int in_full = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const env_f32x4 v = out[c];
          full = full - v[0];
          full = full - v[1];
          full = full - v[2];
          full = full - v[3];
          if (full >= clear) cash = full, in_full = 4 * c + 4;  // (outlays are not negative: never true again once false)
        }
        if ((unsigned)(cl - s0) < (unsigned)in_full) got = (int32_t)mine.k;
        if (in_full == 16) continue;
        // one by one, those that buy nothing (cash < u: the quotient is below 1 and rounds below 1) skipped.
        // The binary32 quotient comes from one binary64 product with the prepared reciprocal of u: the product is
        // within 2^-52 of cash / u, and a quotient of two binary32 numbers is at least 2^-49 (relative) away from
        // every binary32 rounding boundary it does not hit exactly, so the product rounded to binary32 is the
        // correctly rounded cash / u.  It is never negative (cash is not), so truncation is the floor and needs no
        // clamp at 0; the outlay of one share less, (q - 1) u rounded once, is the fused q u - u.
        uint64_t ahead = (0xffffull << s0) & (~0ull << (s0 + in_full));
        while (true) {
          const uint64_t left = affordable(cash, u) & ahead;
          if (left == 0) break;
          const int j = __builtin_ctzll(left);
          const Purchase b = list[c0 + j];
          const float ratio = (float)((double)cash * b.rcp);
          const float q0 = fminf(b.k, truncf(ratio));
          const float out_q = q0 * b.u, out_q1 = fmaf(q0, b.u, -b.u);
          const float bal0 = cash - out_q, bal1 = cash - out_q1;
          const bool over = out_q > cash;
          cash = over ? bal1 : bal0;
          if (cl == j) got = (int32_t)(over ? q0 - 1.0f : q0);
          ahead &= ~1ull << j;
        }
      }
      if (p < total) s_buy[e * lp + p] = got;
    }
  }
  if (live) {
    // -- meanwhile: indicator groups beyond the first NI of a thread (K > 8), and the last DK % 4 indicators
    for (int g = tl + TPE * NI; g < NG; g += TPE) put(g, *reinterpret_cast<const env_f32x4u *>(irow + 4 * g));
  }
  if (live && tl < (DK & 3)) {
    const float v = irow[4 * NG + tl] * d.s_ind;
    o[1 + 2 * D + 4 * NG + tl] = v;
    if (sp) sp[4 * NG + tl] = (__bf16)v;
  }
  __syncthreads();

  // -- executed trades, holdings, account value after them
  double a1 = 0.0;
#pragma unroll
  for (int i = 0; i < ND; ++i) {
    const int dd = tl + TPE * i;
    if (kf[i] > 0.0f) {
      q[i] = s_buy[e * lp + rank[i]];
      h[i] += q[i];
    }
    if (live && dd < D) {
      a1 += (double)h[i] * (double)pv[i];
      const int32_t hn = ri.done ? 0 : h[i];
      s.h[g0 + dd] = hn;
      const float v = (float)hn * d.s_hold;
      o[1 + D + dd] = v;
      if (sp) sp[DK + 1 + D + dd] = (__bf16)v;
      if (io.shares) io.shares[g0 + dd] = q[i];
    }
  }
  a1 = sum_lanes(a1, CW);
  if ((lane & (CW - 1)) == 0) s_part[2 * E + e * 2 + cw] = a1;
  __syncthreads();
  if (live && tl == 0) {
    // -- reward and episode bookkeeping (binary64), reset of the env if its episode ended
    double v0 = (double)cash_in, v1 = (double)cash;
#pragma unroll
    for (int c = 0; c < NCW; ++c) v0 += s_part[e * 2 + c], v1 += s_part[2 * E + e * 2 + c];
    const double r = (v1 - v0) * (double)d.rho;
    double ep = s.ep_ret[n] + r;
    if (ri.done) {
      s.ep_sum[n] += ep;
      s.ep_sqsum[n] += ep * ep;
      s.ep_cnt[n] += 1;
      ep = 0.0;
      cash = d.cash0;
    }
    s.ep_ret[n] = ep;
    s.cash[n] = cash;
    s.tau[n] = ri.done ? start : tau + 1;
    const float v = cash * d.s_cash;
    o[0] = v;
    if (sp) sp[DK] = (__bf16)v;
    io.reward[n] = (float)r;
    io.done[n] = (uint8_t)ri.done;
    if (io.logp) io.logp[n] = fmaf(-0.5f, NCW > 1 ? s_e2[e] : e2, d.logp_const);
  }
}

size_t env_lds(int E, int D) {
  const int D4 = (D + 3) & ~3, lp = D | 1;
  return (size_t)E * lp * sizeof(Purchase) + (size_t)E * (2 * (D4 + 4) + D4 + 20) * 4 + ((size_t)E * lp + 1) * 4 + (size_t)4 * E * 8 +
         (size_t)E * 4 + (size_t)E * 8 * 4;
}

// ------------------------------------------------------------ state plumbing
// *bad = 1 unless every env's episode rows start .. start + H lie inside a table of `rows` rows.
__global__ __launch_bounds__(256) void check_starts_kernel(int32_t N, int32_t H, int32_t rows,
                                                           const int32_t *__restrict__ start, int32_t *bad) {
  int flag = 0;
  for (int i = threadIdx.x; i < N; i += 256) {
    const int32_t s = start[i];
    flag |= (s < 0 || s > rows - 1 - H);
  }
  flag = __syncthreads_or(flag);
  if (threadIdx.x == 0) *bad = flag;
}

__global__ void state_reset_kernel(EnvDims d, EnvState s) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < (size_t)d.N) {
    s.cash[i] = d.cash0;
    s.tau[i] = s.start[i];
    s.ep_ret[i] = 0.0;
    s.ep_sum[i] = 0.0;
    s.ep_sqsum[i] = 0.0;
    s.ep_cnt[i] = 0;
  }
  if (i < (size_t)d.N * d.D) s.h[i] = 0;
}

// user arrays <-> the workspace's
__global__ void state_copy_kernel(EnvDims d, EnvState s, pr_state u, int to_user) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < (size_t)d.N) {
    if (to_user) {
      if (u.cash) u.cash[i] = s.cash[i];
      if (u.cursor) u.cursor[i] = s.tau[i];
      if (u.ep_return) u.ep_return[i] = s.ep_ret[i];
      if (u.ep_sum) u.ep_sum[i] = s.ep_sum[i];
      if (u.ep_sqsum) u.ep_sqsum[i] = s.ep_sqsum[i];
      if (u.ep_count) u.ep_count[i] = s.ep_cnt[i];
    } else {
      if (u.cash) s.cash[i] = u.cash[i];
      if (u.cursor) s.tau[i] = u.cursor[i];
      if (u.ep_return) s.ep_ret[i] = u.ep_return[i];
      if (u.ep_sum) s.ep_sum[i] = u.ep_sum[i];
      if (u.ep_sqsum) s.ep_sqsum[i] = u.ep_sqsum[i];
      if (u.ep_count) s.ep_cnt[i] = u.ep_count[i];
    }
  }
  if (u.holdings && i < (size_t)d.N * d.D) {
    if (to_user)
      u.holdings[i] = s.h[i];
    else
      s.h[i] = u.holdings[i];
  }
}

// -------------------------------------------------------------- leaderboard
// One workgroup per agent: fixed-shape tree reduction (deterministic) of the
// episode statistics of its envs, in binary64.
__global__ __launch_bounds__(256) void leaderboard_reduce_kernel(int32_t envs_per_agent, EnvState s,
                                                                double *__restrict__ mean, double *__restrict__ var) {
  __shared__ double s1[256], s2[256];
  __shared__ long long sc[256];
  const int g = blockIdx.x, tid = threadIdx.x;
  double a = 0.0, b = 0.0;
  long long c = 0;
  for (int i = tid; i < envs_per_agent; i += 256) {
    const size_t n = (size_t)g * envs_per_agent + i;
    a += s.ep_sum[n];
    b += s.ep_sqsum[n];
    c += s.ep_cnt[n];
  }
  s1[tid] = a;
  s2[tid] = b;
  sc[tid] = c;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if (tid < off) {
      s1[tid] += s1[tid + off];
      s2[tid] += s2[tid + off];
      sc[tid] += sc[tid + off];
    }
    __syncthreads();
  }
  if (tid == 0) {
    if (sc[0] > 0) {
      const double m = s1[0] / (double)sc[0];
      mean[g] = m;
      var[g] = s2[0] / (double)sc[0] - m * m;
    } else {
      mean[g] = -INFINITY;
      var[g] = 0.0;
    }
  }
}

// rank[place] = agent id, best mean first, equal means by lower id.
__global__ void leaderboard_rank_kernel(int32_t P, const double *__restrict__ mean, int32_t *__restrict__ rank) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= P) return;
  const double mg = mean[g];
  int place = 0;
  for (int j = 0; j < P; ++j) {
    const double mj = mean[j];
    place += (mj > mg) || (mj == mg && j < g);
  }
  rank[place] = g;
}

}  // namespace

// ------------------------------------------------------------------ launchers

hipError_t launch_observe(hipStream_t st, const EnvDims &d, const EnvState &s, const float *price, const float *ind,
                          float *obs, const ObsShadow &shadow) {
  const int per_block = kThreads / 64;
  hipLaunchKernelGGL(observe_kernel, dim3((d.N + per_block - 1) / per_block), dim3(kThreads), 0, st, d, s, price, ind,
                     obs, shadow);
  return hipGetLastError();
}

template <int E, int ND>
static hipError_t launch_step(hipStream_t st, const EnvDims &d, const EnvState &s, const float *price, const float *ind,
                              const StepIO &io) {
  constexpr auto kern = env_step_kernel<E, ND>;
  const hipError_t e = allow_full_lds<kern>();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)((d.N + E - 1) / E)), dim3(kEnvThreads), env_lds(E, d.D), st, d, s, price, ind, io);
  return hipGetLastError();
}

hipError_t launch_env_step(hipStream_t st, const EnvDims &d, const EnvState &s, const float *price, const float *ind,
                           const StepIO &io) {
  // Half a wavefront per env up to 128 stocks, a whole one up to 256, two beyond; twice as many when all workgroups are
  // then still resident at once, two per compute unit (fewer stocks per thread and an undivided wavefront for the ledger:
  // 512 envs x 60 stocks 8.9 -> 7.4 us, 1024 x 256 13.1 -> 11.3 us; 5000 x 100 would go from 17.5 to 19.7).
  if (d.D <= 32) return launch_step<16, 1>(st, d, s, price, ind, io);
  const bool few8 = d.N <= 8 * 512, few4 = d.N <= 4 * 512;
  if (d.D <= 64) return few8 ? launch_step<8, 1>(st, d, s, price, ind, io) : launch_step<16, 2>(st, d, s, price, ind, io);
  if (d.D <= 128) return few8 ? launch_step<8, 2>(st, d, s, price, ind, io) : launch_step<16, 4>(st, d, s, price, ind, io);
  if (d.D <= 256) return few4 ? launch_step<4, 2>(st, d, s, price, ind, io) : launch_step<8, 4>(st, d, s, price, ind, io);
  if (d.D <= 512) return launch_step<4, 4>(st, d, s, price, ind, io);
  return hipErrorInvalidValue;  // (the networks of this library have at most 512 outputs)
}

hipError_t launch_check_starts(hipStream_t st, int32_t N, int32_t H, int32_t rows, const int32_t *start, int32_t *bad) {
  hipLaunchKernelGGL(check_starts_kernel, dim3(1), dim3(256), 0, st, N, H, rows, start, bad);
  return hipGetLastError();
}

hipError_t launch_state_reset(hipStream_t st, const EnvDims &d, const EnvState &s) {
  const size_t n = (size_t)d.N * (size_t)(d.D > 1 ? d.D : 1);
  hipLaunchKernelGGL(state_reset_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, d, s);
  return hipGetLastError();
}

hipError_t launch_state_copy(hipStream_t st, const EnvDims &d, const EnvState &s, const pr_state &user, bool to_user) {
  const size_t n = (size_t)d.N * (size_t)(d.D > 1 ? d.D : 1);
  hipLaunchKernelGGL(state_copy_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, d, s, user,
                     (int)to_user);
  return hipGetLastError();
}

hipError_t launch_leaderboard(hipStream_t st, int32_t N, int32_t P, const EnvState &s, double *scratch_mean,
                              double *score_mean, double *score_var, int32_t *rank) {
  (void)scratch_mean;
  hipLaunchKernelGGL(leaderboard_reduce_kernel, dim3(P), dim3(256), 0, st, N / P, s, score_mean, score_var);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(leaderboard_rank_kernel, dim3((P + 255) / 256), dim3(256), 0, st, P, score_mean, rank);
  return hipGetLastError();
}

}  // namespace pod
