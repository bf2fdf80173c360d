// Persistent rollout kernel for the few envs of an fp32 network of 256 hidden units:
// one workgroup keeps 16 envs on its compute unit for all T steps (the worker of
// Sec. 4.2; see pod_fused.hip, which has the others).
//
// A step is a chain -- observation, three layers, sample, trade, observation -- and
// while every workgroup has a compute unit to itself everything on it is latency.
// Four wavefronts run the network, a SIMD each, four others the envs, and what depends
// on no decision leaves the chain:
//   network                                   envs (sixteen threads each)
//   layer 1, the portfolio's columns, tanh    reward of step t - 1; request noise and the next market rows
//   --- hidden layer complete, input free
//   layer 2, tanh, output layer               write the market rows of observation t + 1 (records and input tile)
//   --- means complete, hidden tile free
//   layer 1 of step t + 1, market columns     sample, size, trade (pod_trade.h), portfolio columns
//   --- observation t + 1 complete
// The two kinds of wavefront run separate loops with the same barriers: neither's
// registers are live in the other's code.
//
// Bound by the weight stream -- 850 KB a step, which a compute unit takes in at 64 B a
// clock, 5.8 us at 2.3 GHz; 84 KB of layer 2 stay in LDS and the output layer's 48 KB in
// registers (without either 12.3 us a step for 11.4) -- and by the chains beside it: two
// epilogues of 1.1 us, trades 3 us.  301 inputs, per step: 1024 envs 16.2 -> 9.1 us,
// 4096 16.9 -> 11.4 (32 envs on every second compute unit, all eight wavefronts taking
// turns at network and envs); 12 stocks x 4 indicators, 4096 envs, 14.2 -> 8.4.
//
// Compiled with floating-point contraction off (integer decisions depend on
// one rounding per operation).
#include "pod_internal.h"
#include "pod_tile.h"
#include "pod_trade.h"

namespace pod {

namespace {

using namespace tile;
using O = Op<false>;

constexpr int E = 16;               // envs per workgroup
constexpr int NM = 4, NE = 4;       // wavefronts of the network / of the envs
constexpr int NT = 64 * (NM + NE);
constexpr int KBYTES = 2 * O::KBYTES;  // of 32 inputs in an activation row
constexpr int NK2 = 8, HP = tile_pitch<false>(2 * NK2);
constexpr int MUP = 36;             // row pitch of a plane of partial means
constexpr int PLANE = E * MUP;
constexpr int NL = 7;               // units of layer 2 per wavefront that stay in LDS
constexpr int PK = 2, PU = 4 * PK;   // blocks of 32 inputs, and units of weights, in flight per wavefront

using Tr = Trade<E, 2, true, 64 * NE>;
constexpr int TPE = Tr::TPE, ND = 2, ROWS = E / NE;

__host__ __device__ inline int input_pitch(int nkb) { return tile_pitch<false>((nkb + 1) & ~1); }

struct F32Args {
  EnvDims d;
  EnvState st;
  const float *price, *ind;
  PackedNet actor;  // layer 1 in the input order [indicators | prices | holdings | cash], whole blocks of 32 inputs
  int32_t envs_per_agent, T;
  int32_t xpitch;
  const float *noise;  // [T, N, D]
  float *obs;          // [T+1, N, S]
  float *act_raw;      // [T, N, D]
  float *reward;       // [T, N]
  uint8_t *done;       // [T, N]
  float *logp;         // opt [T, N]
  float *mu_out;       // opt [T, N, D]
  int32_t *shares;     // opt [T, N, D]
};

// v_mfma_f32_16x16x32: lane l feeds feature l % 16 and row l % 16, inputs 8 (l / 16) .. + 7 of 32, and holds features
// 4 (l / 16) .. + 3 of row l % 16.  A unit is such an operand of the packed weights, whose blocks are made for 32 features
// and 16 inputs: half the features of two blocks.
__device__ inline void mma16(const Blk3 &w, const Blk3 &x, f32x4 &c) {
#pragma unroll
  for (int i = 0; i < 6; ++i)
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w.p[kSplitA[i]]),
                                                __builtin_bit_cast(bf16x8, x.p[kSplitB[i]]), c, 0, 0, 0);
}

// Where a lane's part of unit 0 lies, in a layer of nct feature tiles, for features from 32 ct on.
__device__ inline const u32x4 *unit_base(const u32x4 *W, int nct, int ct, int lane) {
  return W + ((size_t)(lane >> 5) * nct + ct) * 192 + ((lane >> 4) & 1) * 32 + (lane & 15);
}

// The 64 features of a wavefront are four units per 32 inputs.
// tanh of sixteen values, one operation at a time over all of them (see tanh_in_place).
__device__ inline void tanh_accurate_16(f32x4 (&z)[4]) {
  float e[16], x2[16], ps[16];
  auto all = [&](auto op) {
#pragma unroll
    for (int i = 0; i < 16; ++i) op(i, z[i >> 2][i & 3]);
    __builtin_amdgcn_sched_barrier(0);
  };
  all([&](int i, float x) { e[i] = fabsf(x) * kTwoLog2e; });
  all([&](int i, float) { e[i] = __builtin_amdgcn_exp2f(e[i]); });
  all([&](int i, float x) { x2[i] = x * x; });
  all([&](int i, float) { ps[i] = fmaf(x2[i], 62.0f / 2835.0f, -17.0f / 315.0f); });
  all([&](int i, float) { e[i] = e[i] + 1.0f; });
  all([&](int i, float) { e[i] = __builtin_amdgcn_rcpf(e[i]); });
  all([&](int i, float) { ps[i] = fmaf(x2[i], ps[i], 2.0f / 15.0f); });
  all([&](int i, float) { ps[i] = fmaf(x2[i], ps[i], -1.0f / 3.0f); });
  all([&](int i, float x) { x2[i] = x2[i] * x; });
  all([&](int i, float x) { ps[i] = fmaf(x2[i], ps[i], x); });
  all([&](int i, float x) { e[i] = copysignf(1.0f - 2.0f * e[i], x); });
  all([&](int i, float x) { z[i >> 2][i & 3] = fabsf(x) < 0.25f ? ps[i] : e[i]; });
}

__device__ inline void fetch_unit(Blk3 &b, const u32x4 *W, int u) {
  fetch_w(b, W + (size_t)(u >> 2) * (2 * 8 * 192) + ((u >> 1) & 1) * 192 + (u & 1) * 16);
}

// acc += inputs 32 [0, n) of a range; the ring holds the first units.  N > 0: n at compile time, in straight-line code.
template <int N>
__device__ inline void products(f32x4 (&acc)[4], Blk3 (&ring)[PU], const unsigned char *x, const u32x4 *W, int n) {
  if constexpr (N > 0) {
    Blk3 xn;
    fetch_x(xn, x);
#pragma unroll
    for (int K = 0; K < N; ++K) {
      const Blk3 xv = xn;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int u = 4 * K + j;
        if (j == 0 && K + 1 < N) {
          fetch_x(xn, x + (K + 1) * KBYTES);
          __builtin_amdgcn_sched_barrier(0);
        }
        mma16(ring[u % PU], xv, acc[j]);
        if (u + PU < 4 * N) fetch_unit(ring[u % PU], W, u + PU);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  } else {
    auto block = [&](int K, int k) {  // (k: K modulo PK, at compile time)
      Blk3 xv;
      fetch_x(xv, x + K * KBYTES);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        mma16(ring[4 * k + j], xv, acc[j]);
        fetch_unit(ring[4 * k + j], W, 4 * min(K + PK, n - 1) + j);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    int K = 0;
    for (; K + PK <= n; K += PK) {
#pragma unroll
      for (int k = 0; k < PK; ++k) block(K + k, k);
    }
#pragma unroll
    for (int k = 0; k < PK - 1; ++k)
      if (K + k < n) block(K + k, k);
  }
}

// Layer 2: the first NL units from LDS (`own`, this lane's), the others through the ring, which holds the first of them.
__device__ inline void products2(f32x4 (&acc)[4], Blk3 (&ring)[PU], const unsigned char *x, const u32x4 *own, const u32x4 *W) {
  Blk3 xn, wn;
  fetch_x(xn, x);
  fetch_w(wn, own);
#pragma unroll
  for (int K = 0; K < NK2; ++K) {
    const Blk3 xv = xn;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int u = 4 * K + j, r = u - NL;
      const Blk3 wv = r < 0 ? wn : ring[r < 0 ? 0 : r % PU];
      if (j == 0 && K + 1 < NK2) fetch_x(xn, x + (K + 1) * KBYTES);
      if (u + 1 < NL) fetch_w(wn, own + (u + 1) * 192);
      __builtin_amdgcn_sched_barrier(0);
      mma16(wv, xv, acc[j]);
      if (r >= 0 && u + PU < 4 * NK2) fetch_unit(ring[r % PU], W, u + PU);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// NK1, NH: 32-input blocks of layer 1, and how many of them hold market columns only (0: at run time)
template <int NK1, int NH>
__global__ __launch_bounds__(NT, 2) void rollout_f32_kernel(F32Args a) {
  extern __shared__ __align__(16) unsigned char lds[];
  const EnvDims &d = a.d;
  const int D = d.D, DK = D * d.K, S = d.S;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n0 = (int)xcd_index(blockIdx.x, gridDim.x) * E;
  const size_t N = (size_t)d.N;
  unsigned char *ldsX = lds, *ldsH = ldsX + E * a.xpitch;  // input tile; hidden tile, and in it the trades' scratch
  float *planes = reinterpret_cast<float *>(ldsH + E * HP);  // [NM][E][MUP] partial means
  float *ldsBias = planes + NM * PLANE;                     // b1 | b2 | b3
  double *ldsTerms = reinterpret_cast<double *>(ldsBias + 2 * 256 + 32);  // holdings' values, read while the hidden tile is in use
  u32x4 *ldsW = reinterpret_cast<u32x4 *>(ldsTerms + E * 32);
  const Net net = net_of(a.actor, (n0 % d.N) / a.envs_per_agent);

  for (int i = tid; i < E * a.xpitch / 4; i += NT) reinterpret_cast<uint32_t *>(ldsX)[i] = 0u;  // (padded k columns stay so)
  stage_net<NT>(net, ldsBias, nullptr, tid);
  __syncthreads();

  if (w < NM) {
    // ---------------------------------------------------------------- the network, features 64 w ..
    const int nk1 = NK1 > 0 ? NK1 : net.nkb[0] / 2, nh = NH > 0 ? NH : (DK + D) / 32;
    const int row = lane & 15, kq = lane >> 4;
    const unsigned char *xrow = ldsX + row * a.xpitch + O::HALF * kq, *hrow = ldsH + row * HP + O::HALF * kq;
    Blk3 ring[PU];
    f32x4 acc[4];
    auto prime_range = [&](const u32x4 *W, int n) {
#pragma unroll
      for (int u = 0; u < PU; ++u)
        if (u / 4 < n) fetch_unit(ring[u], W, u);
    };
    auto clear = [&]() {
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    };
    auto activate = [&](const float *bias) {
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j] += *reinterpret_cast<const f32x4 *>(bias + 64 * w + 16 * j + 4 * kq);
      tanh_accurate_16(acc);
    };
    int lane_s = lane;
    const u32x4 *W1, *W2;
    auto addresses = [&]() {  // (opaque per step, or the addresses of all weight blocks are kept across the steps)
      asm volatile("" : "+v"(lane_s));
      W1 = unit_base(net.W[0], 8, 2 * w, lane_s);
      W2 = unit_base(net.W[1], 8, 2 * w, lane_s);
    };
    auto head = [&]() {
      clear();
      products<NH>(acc, ring, xrow, W1, nh);
      prime_range(W1 + (size_t)nh * (2 * 8 * 192), nk1 - nh);
    };
    addresses();
    // kept: the first units of layer 2 (LDS) and the output layer's weights (registers).  A lane of that layer's operand
    // takes the two halves of its piece from the places the order of its inputs has them in (see below).
    u32x4 *own = ldsW + (size_t)w * (NL * 192) + lane;
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      Blk3 b;
      fetch_unit(b, W2, u);
#pragma unroll
      for (int i = 0; i < 3; ++i) own[u * 192 + 64 * i] = b.p[i];
    }
    const unsigned char *W3 = reinterpret_cast<const unsigned char *>(net.W[2] + (size_t)w * (4 * 192) + (kq >> 1) * 32 + row) + 8 * (kq & 1);
    Blk3 w3[2][2];
#pragma unroll
    for (int K = 0; K < 2; ++K)
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          const u32x2 lo = *reinterpret_cast<const u32x2 *>(W3 + (K * 384 + c * 16 + i * 64) * 16);
          const u32x2 hi = *reinterpret_cast<const u32x2 *>(W3 + (K * 384 + 192 + c * 16 + i * 64) * 16);
          w3[K][c].p[i] = u32x4{lo[0], lo[1], hi[0], hi[1]};
        }
    prime_range(W1, nh);
    __syncthreads();  // observation 0 complete
    head();
    for (int t = 0; t < a.T; ++t) {
      __syncthreads();  // observation t complete
      products<NK1 - NH>(acc, ring, xrow + nh * KBYTES, W1 + (size_t)nh * (2 * 8 * 192), nk1 - nh);
      addresses();
#pragma unroll
      for (int u = 0; u < PU; ++u) fetch_unit(ring[u], W2, NL + u);
      activate(ldsBias);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        O::store4<true>(ldsH + row * HP + O::off(64 * w + 16 * j + 4 * kq), acc[j][0], acc[j][1], acc[j][2], acc[j][3]);
      __syncthreads();  // first hidden layer complete, input tile free
      clear();
      products2(acc, ring, hrow, own, W2);
      // Output layer, from registers: the eight values a lane holds of 32 features are an operand of the transposed product
      // in another order of its inputs.  Each wavefront adds up its own features for all outputs.
      prime_range(W1, nh);
      activate(ldsBias + 256);
      f32x4 o[2][2];  // (one sum over both halves leaves a larger error: 3.16e-7 in the 2-norm of the means for 3.06e-7)
#pragma unroll
      for (int K = 0; K < 2; ++K) {
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = acc[2 * K + (i >> 2)][i & 3];
        bf16x8 xs[3];
        split3<true>(v, xs);
        Blk3 xv;
#pragma unroll
        for (int i = 0; i < 3; ++i) xv.p[i] = __builtin_bit_cast(u32x4, xs[i]);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          o[K][c] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
          mma16(w3[K][c], xv, o[K][c]);
        }
      }
#pragma unroll
      for (int c = 0; c < 2; ++c) *reinterpret_cast<f32x4 *>(planes + w * PLANE + row * MUP + 16 * c + 4 * kq) = o[0][c] + o[1][c];
      __syncthreads();  // means and the market columns of observation t + 1 complete
      if (t + 1 < a.T) head();
    }
    return;
  }

  // ------------------------------------------------------------------ the envs
  __builtin_amdgcn_s_setprio(3);
  Tr trade(ldsH, D);
  trade.terms = ldsTerms;
  const int et = tid - 64 * NM, e = et / TPE, tl = et & (TPE - 1), ew = w - NM;
  const int n = n0 + e;
  const float *lb3 = ldsBias + 2 * 256;
  int32_t tau = a.st.tau[n];
  const int32_t start = a.st.start[n];
  float cash = a.st.cash[n];
  double ep_ret = a.st.ep_ret[n], ep_sum = a.st.ep_sum[n], ep_sqsum = a.st.ep_sqsum[n];
  int32_t ep_cnt = a.st.ep_cnt[n];
  int32_t h[ND];
  float pn[ND];
  int dd[ND];
#pragma unroll
  for (int i = 0; i < ND; ++i) dd[i] = min(tl + TPE * i, D - 1);  // (stocks behind the last: that one again, not used)
  auto mine = [&](int i) { return tl + TPE * i < D; };
  unsigned char *xenv = ldsX + e * a.xpitch;
  const int li = min(lane, (DK >> 2) - 1), lp = min(lane, D - 1);
  // market part of an observation: a row per instruction, prices and 16-byte groups of indicators (lanes beyond them, and
  // with few groups, repeat the last one)
  float r_p[ROWS];
  f32x4 r_i[ROWS];
  auto fetch_market = [&](int32_t row) {
#pragma unroll
    for (int j = 0; j < ROWS; ++j) {
      const size_t ro = (size_t)__builtin_amdgcn_readlane(row, TPE * j);
      r_p[j] = __builtin_nontemporal_load(&a.price[ro * D + lp]);
      r_i[j] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(a.ind + ro * DK) + li);
    }
  };
  auto emit_market = [&](float *obs) {
#pragma unroll
    for (int j = 0; j < ROWS; ++j) {
      const int er = ROWS * ew + j;
      float *orow = obs + (size_t)(n0 + er) * S;
      unsigned char *x = ldsX + er * a.xpitch;
      const float pv = r_p[j] * d.s_price;
      __builtin_nontemporal_store(pv, &orow[1 + lp]);
      O::store1(x + O::off(DK + lp), pv);
      f32x4 v = r_i[j];
      v[0] *= d.s_ind, v[1] *= d.s_ind, v[2] *= d.s_ind, v[3] *= d.s_ind;
      // observation rows are 4-byte aligned only; a 16-byte store needs no more than that
      __builtin_nontemporal_store(v, reinterpret_cast<f32x4 *>(orow + 1 + 2 * D) + li);
      O::store4(x + O::off(4 * li), v[0], v[1], v[2], v[3]);
    }
  };
  auto put_holding = [&](float *obs, int i) {
    const float v = (float)h[i] * d.s_hold;
    __builtin_nontemporal_store(v, &obs[(size_t)n * S + 1 + D + dd[i]]);
    O::store1(xenv + O::off(DK + D + dd[i]), v);
  };
  auto put_cash = [&](float *obs) {
    if (tl == 0) {
      const float v = cash * d.s_cash;
      __builtin_nontemporal_store(v, &obs[(size_t)n * S]);
      O::store1(xenv + O::off(DK + 2 * D), v);
    }
  };
  {
    const int32_t row = tau * d.M + (d.M == 1 ? 0 : n);
    fetch_market(row);
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      h[i] = a.st.h[(size_t)n * D + dd[i]];
      pn[i] = a.price[(size_t)row * D + dd[i]];
    }
    emit_market(a.obs);
#pragma unroll
    for (int i = 0; i < ND; ++i)
      if (mine(i)) put_holding(a.obs, i);
    put_cash(a.obs);
  }
  __syncthreads();  // observation 0 complete
#pragma unroll
  for (int i = 0; i < ND; ++i) trade.put_term(i, mine(i) ? (double)h[i] * (double)pn[i] : 0.0);
  double value = trade.value(cash);  // the account's, before the next trades
  float e2 = 0.0f, cash_after = cash;
  int32_t ended = 0;
  // Reward and episode sums of step t (binary64), beside the next step's first phase: no observation needs them.
  auto settle = [&](int t) {
    const double after = trade.value(cash_after), r = (after - value) * (double)d.rho;
    value = ended ? (double)d.cash0 : after;
    ep_ret += r;
    if (ended) {
      ep_sum += ep_ret;
      ep_sqsum += ep_ret * ep_ret;
      ep_cnt += 1;
      ep_ret = 0.0;
    }
    if (tl == 0) {
      const size_t tn = (size_t)t * N + n;
      a.reward[tn] = (float)r;
      a.done[tn] = (uint8_t)ended;
      if (a.logp) a.logp[tn] = fmaf(-0.5f, e2, d.logp_const);
    }
  };
  for (int t = 0; t < a.T; ++t) {
    __syncthreads();  // observation t complete
    const size_t g0 = ((size_t)t * N + n) * D;
    float *obs_next = a.obs + (size_t)(t + 1) * N * S;
    const RowInfo ri = rows_of(d, tau, start, n);
    float eps[ND], pv[ND], po[ND];
    fetch_market(ri.row_obs);
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      eps[i] = __builtin_nontemporal_load(a.noise + g0 + dd[i]);
      pv[i] = a.price[(size_t)ri.row_val * D + dd[i]];
      po[i] = a.price[(size_t)ri.row_obs * D + dd[i]];
    }
    if (t > 0) settle(t - 1);
    const typename Tr::Unit units = Tr::unit_of(d, pn);
    __syncthreads();  // input tile free
    emit_market(obs_next);
    __syncthreads();  // means complete, the hidden tile is free
    float a_raw[ND], mu[ND];
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      const float *m = planes + e * MUP + dd[i];
      mu[i] = finish_out((m[0] + m[PLANE]) + (m[2 * PLANE] + m[3 * PLANE]), lb3[dd[i]], 1);
      a_raw[i] = mu[i] + d.sigma * eps[i];  // two roundings (contraction is off)
    }
    int32_t q[ND];
    double unused;
    trade.run(
        d, true, a_raw, eps, pn, units, pv, h, q, cash, unused, e2, a.logp != nullptr, []() {},
        [&]() {
#pragma unroll
          for (int i = 0; i < ND; ++i)
            if (mine(i)) {
              __builtin_nontemporal_store(a_raw[i], &a.act_raw[g0 + dd[i]]);
              if (a.mu_out) a.mu_out[g0 + dd[i]] = mu[i];
            }
        },
        [&](int i) {
          if (ri.done) h[i] = 0;
          put_holding(obs_next, i);
          if (a.shares) a.shares[g0 + dd[i]] = q[i];
        });
    cash_after = cash;
    ended = ri.done;
    if (ended) cash = d.cash0;
    tau = ended ? start : tau + 1;
#pragma unroll
    for (int i = 0; i < ND; ++i) pn[i] = po[i];
    put_cash(obs_next);
  }
  settle(a.T - 1);
#pragma unroll
  for (int i = 0; i < ND; ++i)
    if (mine(i)) a.st.h[(size_t)n * D + dd[i]] = h[i];
  if (tl == 0) {
    a.st.tau[n] = tau;
    a.st.cash[n] = cash;
    a.st.ep_ret[n] = ep_ret;
    a.st.ep_sum[n] = ep_sum;
    a.st.ep_sqsum[n] = ep_sqsum;
    a.st.ep_cnt[n] = ep_cnt;
  }
}

}  // namespace

// Up to a workgroup for each of the 256 compute units; with two rounds of them, 32 envs per workgroup take as long (8192 envs
// 20.4 us a step against 20.7, 16384 37.9 against 39.5, 5120 17.5 against 20.7).
bool fused_few_envs(const pr_config &c) { return c.mlp_dtype == PR_MLP_F32 && c.n_envs <= 256 * E; }

// LDS of the kernel; the input tile has whole blocks of 32 inputs.
size_t fused_f32_lds_bytes(const pr_config &c) {
  const int S = 1 + 2 * c.n_stocks + c.n_stocks * c.n_ind;
  return (size_t)E * (input_pitch((S + 15) / 16) + HP) + ((size_t)NM * PLANE + (2 * 256 + 32)) * 4 + (size_t)E * 32 * 8 + (size_t)NM * NL * 3072;
}

hipError_t launch_rollout_fused_f32(hipStream_t st, const pr_config &c, const EnvDims &d, const EnvState &s,
                                    const float *price, const float *ind, const PackedNet &actor, int32_t envs_per_agent,
                                    int32_t T, const float *noise, const pr_buffers &out) {
  F32Args a;
  a.d = d, a.st = s, a.price = price, a.ind = ind, a.actor = actor, a.envs_per_agent = envs_per_agent, a.T = T;
  a.xpitch = input_pitch(actor.nkb[0]);
  a.noise = noise, a.obs = out.obs, a.act_raw = out.act_raw, a.reward = out.reward, a.done = out.done, a.logp = out.logp;
  a.mu_out = out.mu, a.shares = out.shares;
  if (actor.bf16 || actor.nkb[0] % 2 || actor.nkb[1] != 2 * NK2 || actor.nct[0] != 8 || actor.nct[2] != 1 || d.N % E || envs_per_agent % E)
    return hipErrorInvalidValue;
  const size_t lds = fused_f32_lds_bytes(c);
  if (trade_lds(E, true, d.D) > (size_t)E * HP || lds > (size_t)kMaxLdsBytes) return hipErrorInvalidValue;
  auto launch = [&](auto nk1, auto nh) {
    constexpr auto kern = rollout_f32_kernel<decltype(nk1)::value, decltype(nh)::value>;
    const hipError_t e = allow_full_lds<kern>();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)(d.N / E)), dim3(NT), lds, st, a);
    return hipGetLastError();
  };
  if (actor.nkb[0] == 20 && (d.D * d.K + d.D) / 32 == 8) return launch(std::integral_constant<int, 10>{}, std::integral_constant<int, 8>{});
  return launch(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
}

}  // namespace pod
