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
#include "pod_trade.h"

namespace pod {

namespace {

constexpr int kThreads = 256;

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
// One launch per step: 512 threads step E envs (the trades: pod_trade.h).  IND: the next observation's indicators too.  The cursor is read by every thread of an env (no
// barrier in front of the prices), the market part of the next observation is requested together with the prices and
// written while the orders are packed.
// Measured per step (kernel trace): 2048 envs x 500 stocks x 4 indicators 106 -> 22 us, 5000 x 100 x 8 30.2 -> 18.6,
// 16384 x 100 x 8 60 -> 37, 4096 x 30 x 8 12.3 -> 7.1, 16384 x 30 x 8 17.0 -> 15.5, 16 x 5 x 2 6.0 -> 3.8 (before: order
// slots of up to 32 envs and a ledger over all of them in LDS, holdings stored stock-major and hence moved in short
// runs).  The bytes of the first of these take 10 us.
template <int E, int ND, bool IND>
__global__ __launch_bounds__(kEnvThreads, 4) void env_step_kernel(EnvDims d, EnvState s, const float *__restrict__ price,
                                                                 const float *__restrict__ ind, StepIO io) {
  using Tr = Trade<E, ND, false>;
  constexpr int TPE = Tr::TPE;         // threads per env
  constexpr int NI = ND == 1 ? 4 : 8;  // 16-byte indicator groups per thread that are requested with the prices
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const int D = d.D, DK = D * d.K;
  const int tid = threadIdx.x;
  const int e = tid / TPE, tl = tid & (TPE - 1);
  const int n0 = blockIdx.x * E, n = min(n0 + e, d.N - 1);
  const bool live = n0 + e < d.N;

  // -- requests that depend on nothing
  const int32_t tau = s.tau[n], start = s.start[n];
  const float cash_in = s.cash[n];
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
  env_f32x4 iv[NI];
#pragma unroll
  for (int j = 0; j < NI; ++j) {
    const int g = tl + TPE * j;
    if (IND && g < NG) iv[j] = *reinterpret_cast<const env_f32x4u *>(irow + 4 * g);
  }

  float *o = io.obs_next + (size_t)n * d.S;
  __bf16 *sp = io.shadow.p ? reinterpret_cast<__bf16 *>(io.shadow.p) + (size_t)n * io.shadow.pitch : nullptr;
  auto put = [&](int g, env_f32x4 v) {
    v[0] *= d.s_ind, v[1] *= d.s_ind, v[2] *= d.s_ind, v[3] *= d.s_ind;
    __builtin_nontemporal_store(v, reinterpret_cast<env_f32x4u *>(o + 1 + 2 * D + 4 * g));
    if (sp) {
      typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
      *reinterpret_cast<bf16x4 *>(sp + 4 * g) = bf16x4{(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
    }
  };
  float a_raw[ND];
#pragma unroll
  for (int i = 0; i < ND; ++i) {
    const int dd = tl + TPE * i;
    a_raw[i] = mu[i] + d.sigma * eps[i];  // two roundings (contraction is off)
    if (live && dd < D) io.act_raw[g0 + dd] = a_raw[i];
  }
  Tr trade(lds_raw, D);
  int32_t q[ND];
  float cash = cash_in, e2;
  double r;
  trade.run(
      d, live, a_raw, eps, pn, Tr::unit_of(d, pn), pv, h, q, cash, r, e2, io.logp != nullptr,
      [&]() {
        // market part of the next observation
#pragma unroll
        for (int i = 0; i < ND; ++i) {
          const int dd = tl + TPE * i;
          if (live && dd < D) {
            const float v = po[i] * d.s_price;
            o[1 + dd] = v;
            if (sp) sp[DK + 1 + dd] = (__bf16)v;
          }
        }
        if (IND && live) {
#pragma unroll
          for (int j = 0; j < NI; ++j) {
            const int g = tl + TPE * j;
            if (g < NG) put(g, iv[j]);
          }
        }
      },
      [&]() {
        // indicator groups beyond the first NI of a thread (K > 8), and the last DK % 4 indicators
        if (IND && live) {
          for (int g = tl + TPE * NI; g < NG; g += TPE) put(g, *reinterpret_cast<const env_f32x4u *>(irow + 4 * g));
          if (tl < (DK & 3)) {
            const float v = irow[4 * NG + tl] * d.s_ind;
            o[1 + 2 * D + 4 * NG + tl] = v;
            if (sp) sp[4 * NG + tl] = (__bf16)v;
          }
        }
      },
      [&](int i) {
        // executed trades and holdings, cleared when the episode ended
        const int dd = tl + TPE * i;
        const int32_t hn = ri.done ? 0 : h[i];
        s.h[g0 + dd] = hn;
        const float v = (float)hn * d.s_hold;
        o[1 + D + dd] = v;
        if (sp) sp[DK + 1 + D + dd] = (__bf16)v;
        if (io.shares) io.shares[g0 + dd] = q[i];
      });
  if (live && tl == 0) {
    // -- episode bookkeeping (binary64), reset of the env if its episode ended
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
    if (io.logp) io.logp[n] = fmaf(-0.5f, e2, d.logp_const);
  }
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

template <int E, int ND, bool IND>
static hipError_t launch_step_inst(hipStream_t st, const EnvDims &d, const EnvState &s, const float *price, const float *ind,
                                   const StepIO &io) {
  constexpr auto kern = env_step_kernel<E, ND, IND>;
  const hipError_t e = allow_full_lds<kern>();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)((d.N + E - 1) / E)), dim3(kEnvThreads), trade_lds(E, false, d.D), st, d, s, price, ind, io);
  return hipGetLastError();
}

template <int E, int ND>
static hipError_t launch_step(hipStream_t st, const EnvDims &d, const EnvState &s, const float *price, const float *ind,
                              const StepIO &io) {
  return io.ind_done ? launch_step_inst<E, ND, false>(st, d, s, price, ind, io) : launch_step_inst<E, ND, true>(st, d, s, price, ind, io);
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
