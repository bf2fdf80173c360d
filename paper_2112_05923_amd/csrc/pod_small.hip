// The stepwise schedule's rollout for small networks: one launch for all T steps.
//
// With 64 or 128 hidden units a step is a few microseconds of launches around a
// few hundred nanoseconds of work: 17 us for 16 envs, whatever the device does.
// Envs are independent, so a workgroup keeps 16 of them, their state and the
// WHOLE policy network on its compute unit instead: the weights stay in registers
// from the first step to the last, the observation lives in LDS as the operand
// layer 1 reads, and only the rollout's records go to memory.
//
// What bounds a step is latency: three layers, each one product and one barrier, then
// the trades' chain (pod_trade.h).  A wavefront owns 16 features of a layer with all of
// their inputs (16 x 16 x 32 instructions: the 16 envs fill their columns); partial sums
// over k-blocks, which went through LDS with a barrier of their own, took as long again
// (16 envs x 5 stocks, 64 steps with values 239 -> 207 us).  With up to 16 stocks half of the
// wavefronts are enough to trade, and the others move the market, prepare the next quotes and
// keep the books of the step before meanwhile (207 -> 152; with 30 stocks and four wavefronts
// the trades themselves take longer than that saves: 512 envs x 30 x 8 333 -> 341).  The loads
// of a step -- noise, the next market row -- depend on the cursor only and travel behind the
// network.
// Per step, first (a network launch or three and an env launch) -> in one launch -> now:
//   fp32,  64 hidden units: 16 envs x 5 stocks 19.6 -> 3.5 -> 2.1 us, 512 x 30 x 8 indicators 30 -> 5.1 -> 4.5
//   fp32, 128: 64 x 10 x 2 27 -> 5.3 -> 2.9, 512 x 30 x 8 37 -> 10.9 -> 7.0 (57 registers spill; 129 before)
//   bf16, 128: 512 x 30 x 8 30 -> 4.0 -> 3.2
#include <algorithm>

#include "pod_internal.h"
#include "pod_tile.h"
#include "pod_trade.h"

namespace pod {
namespace {

using tile::f32x16;
using tile::f32x4;
using tile::u32x2;
using tile::u32x4;

constexpr int SE = 16;            // envs per workgroup
constexpr int kWaves = 8;
constexpr int kMaxBlocks = 20;    // k-blocks of layer 1: up to 320 inputs

struct SmallArgs {
  EnvDims d;
  EnvState st;
  const float *price, *ind;
  PackedNet net;  // layer 1 in the input order [indicators | cash | prices | holdings]
  int32_t envs_per_agent, T;
  int32_t runs;        // an XCD takes a run of workgroups
  const float *noise;  // [T, N, D]
  float *obs;          // [T+1, N, S]
  float *act_raw;      // [T, N, D]
  float *reward;       // [T, N]
  uint8_t *done;       // [T, N]
  float *logp;         // opt [T, N]
  float *mu;           // opt [T, N, D]
  int32_t *shares;     // opt [T, N, D]
};

// What a chain of products with the 16 envs adds up to; fp32: the three smallest of the six in a sum of their own (mma16).
struct Sums {
  f32x4 hi = {0.0f, 0.0f, 0.0f, 0.0f}, lo = {0.0f, 0.0f, 0.0f, 0.0f};
};

template <int HD>
struct Geometry {
  static constexpr int TILES = HD / 16;       // feature tiles of a hidden layer
  static constexpr int WT = kWaves / TILES;   // wavefronts that share one
  static constexpr int F = 4 / WT;            // features of a lane that its wavefront takes through tanh
  static constexpr int KS = HD / 32;          // k-steps of layers 2 and 3
};
// Which kernels do not request the k-blocks behind the last one.  The others request the last one in their place and replace it by
// zeros, for which the weights are waited for before the state and the market's first row are requested: a call of one step, fp32, 64
// units, us without values 16 envs x 12 stocks x 4 9.0 -> 8.6, 500 x 16 x 8 11.7 -> 10.6, 10000 x 20 x 7 35.4 -> 32.2; 128 units, 500 x 12 x 4
// 10.8 -> 9.6; with values 4096 x 20 x 7, 64 units 26.3 -> 23.5.  But they have more registers to spill in fp32 with 128 units and more than
// 160 inputs (4096 x 30 x 8, 32 steps 272 -> 294 us), and in bf16 it pays with many blocks only (4096 x 12 x 4, 128 units, 32 steps with
// values 124 -> 127).
constexpr bool skips_blocks(bool bf16, int hd, int ks1) { return bf16 ? ks1 == 10 : hd == 64 || ks1 < 10; }

constexpr int kMeanPitch = 36, kSharePitch = 66;  // floats: partial means of an env; a wavefront's sums of a feature

// What a step's trades need of a stock's price, in LDS.
struct __attribute__((aligned(16))) Quote {
  float price, cost;  // and the unit cost of a purchase
  double rcp;         // 1 / cost
};

inline size_t small_lds(int KS, bool split, bool apart, int xpitch, int hpitch, int D) {
  return (size_t)SE * (xpitch + 2 * hpitch) + (size_t)KS * SE * kMeanPitch * 4 + (split ? (size_t)kWaves * 2 * kSharePitch * 4 : 0) +
         (apart ? 2 * (size_t)SE * (D | 1) * sizeof(Quote) + 2 * SE * 4 : 0) + trade_lds(SE, true, D) +
         (apart ? (size_t)SE * ((D + 3) & ~3) * 8 : 0);
}

// HD: hidden units; KS1: k-steps (of 32 inputs) of layer 1; SPLIT: the two wavefronts of a feature tile take half of them each;
// APART: four wavefronts trade, with 16 threads to an env, and the others move the market and keep the books beside them; or all
// eight do all of it, 32 threads to an env
template <bool BF16, int HD, int KS1, bool SPLIT, bool APART>
__global__ __launch_bounds__(kEnvThreads, 2) void rollout_small_kernel(SmallArgs a) {
  using namespace tile;
  using O = Op<BF16>;
  using Block = typename O::Block;
  using Gm = Geometry<HD>;
  // where the weights leave few registers, what follows from the thread's index is formed anew in every step
  // (512 envs x 30 stocks x 8, 128 units, 64 steps 604 -> 504 us; 64 units, which spill ten registers without it, 337 -> 348)
  constexpr bool TIGHT = !BF16 && HD == 128 && KS1 > 2;
  using Tr = Trade<SE, 1, true, APART ? kEnvThreads / 2 : kEnvThreads, TIGHT>;
  constexpr int TPE = Tr::TPE, NI = 4, F = Gm::F, KS = Gm::KS, NCT = HD / 32, NP = 64 * kPlanes<Block>;
  static_assert(!SPLIT || (Gm::WT == 2 && KS1 % 2 == 0), "");
  constexpr int B1 = SPLIT ? KS1 / 2 : KS1;
  constexpr int XP = tile_pitch<BF16>(2 * KS1), HP = tile_pitch<BF16>(2 * KS);
  extern __shared__ __align__(16) unsigned char lds[];
  const EnvDims &d = a.d;
  const int D = d.D, DK = D * d.K, S = d.S, NG = DK / 4, D4 = (D + 3) & ~3, QP = D | 1;
  unsigned char *ldsX = lds, *ldsH1 = ldsX + SE * XP, *ldsH2 = ldsH1 + SE * HP;
  float *means = reinterpret_cast<float *>(ldsH2 + SE * HP);  // [KS][SE][kMeanPitch]
  float *share = means + KS * SE * kMeanPitch;                // SPLIT: [kWaves][2][kSharePitch]
  // APART, by the step's parity: [2][SE][QP], [2][SE] cash after the trades, and a second set of the trades' terms
  Quote *quotes = reinterpret_cast<Quote *>(share + (SPLIT ? kWaves * 2 * kSharePitch : 0));
  float *balance = reinterpret_cast<float *>(quotes + (APART ? 2 * SE * QP : 0));
  Tr trade(reinterpret_cast<unsigned char *>(balance + (APART ? 2 * SE : 0)), D);
  double *const terms0 = trade.terms;
  auto terms_of = [&](int t) { trade.terms = APART ? terms0 + (t & 1) * SE * D4 : terms0; };

  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool trader = !APART || w < kWaves / 2, keeper = !APART || !trader;
  int e = trade.thread() / TPE, tl = tid & (TPE - 1);  // of either kind: its env, its lane of the env
  const int dd = min(tl, D - 1);
  const int n0 = (int)(a.runs ? xcd_run(blockIdx.x, gridDim.x) : blockIdx.x) * SE, n = min(n0 + e, d.N - 1);
  const bool live = n0 + e < d.N, own = live && tl < D;
  const size_t N = (size_t)d.N;

  // -- the network: this wavefront's weight blocks, this lane's biases
  const Net net = net_of(a.net, (n0 % d.N) / a.envs_per_agent);
  const int ft = w % Gm::TILES, wt = w / Gm::TILES;  // feature tile of layers 1 and 2, and which of its wavefronts this is
  const int ot = w & 1, ok = w >> 1;                 // output tile and k-step of layer 3
  const int q4 = lane >> 4, row = lane & 15;
  // (packed blocks are 32 features x 16 inputs)
  auto fetch = [&](Block &b, const u32x4 *W, int nct, int nkb, int tile, int ks) {
    const int kb = 2 * ks + (q4 >> 1);
    if constexpr (skips_blocks(BF16, HD, KS1)) {
      b = Block{};
      if (kb < nkb) fetch_w(b, W + ((size_t)kb * nct + (tile >> 1)) * NP + (tile & 1) * 16 + row + 32 * (q4 & 1));
    } else {
      fetch_w(b, W + ((size_t)min(kb, nkb - 1) * nct + (tile >> 1)) * NP + (tile & 1) * 16 + row + 32 * (q4 & 1));
      if (kb >= nkb) b = Block{};
    }
  };
  Block w1[B1], w2[KS], w3;
#pragma unroll
  for (int i = 0; i < B1; ++i) fetch(w1[i], net.W[0], NCT, net.nkb[0], ft, SPLIT ? wt * B1 + i : i);
#pragma unroll
  for (int i = 0; i < KS; ++i) fetch(w2[i], net.W[1], NCT, 2 * KS, ft, i);
  fetch(w3, net.W[2], 1, 2 * KS, ot, min(ok, KS - 1));
  const int f0 = 16 * ft + 4 * q4 + F * wt;  // the first of this lane's features of env `row`
  float bias1[F], bias2[F];
#pragma unroll
  for (int i = 0; i < F; ++i) bias1[i] = net.b[0][f0 + i], bias2[i] = net.b[1][f0 + i];
  const float bias3 = net.b[2][tl];

  // -- state: of the traders cash and holdings, of the others the books
  int32_t tau = a.st.tau[n];
  const int32_t start = a.st.start[n];
  float cash = a.st.cash[n];
  int32_t h[1] = {a.st.h[(size_t)n * D + dd]};
  double ep_ret = a.st.ep_ret[n], ep_sum = a.st.ep_sum[n], ep_sqsum = a.st.ep_sqsum[n];
  int32_t ep_cnt = a.st.ep_cnt[n];

  auto xrow = [&](int byte) { return ldsX + e * XP + byte; };
  float *orow = a.obs + (size_t)n * S;  // of the observation being written
  auto put_ind = [&](int g, env_f32x4 v) {
    v[0] *= d.s_ind, v[1] *= d.s_ind, v[2] *= d.s_ind, v[3] *= d.s_ind;
    *reinterpret_cast<env_f32x4u *>(orow + 1 + 2 * D + 4 * g) = v;
    O::store4(xrow(O::off(4 * g)), v[0], v[1], v[2], v[3]);
  };
  auto put_price = [&](float p) {
    const float v = p * d.s_price;
    orow[1 + tl] = v;
    O::store1(xrow(O::off(DK + 1 + tl)), v);
  };
  auto quote = [&](float p, int par) {
    const float u = p * d.one_plus_c;
    quotes[(par * SE + e) * QP + tl] = Quote{p, u, 1.0 / (double)u};
  };
  auto put_holding = [&](int32_t x) {
    const float v = (float)x * d.s_hold;
    orow[1 + D + tl] = v;
    O::store1(xrow(O::off(DK + 1 + D + tl)), v);
  };
  auto put_cash = [&](float c) {
    const float v = c * d.s_cash;
    orow[0] = v;
    O::store1(xrow(O::off(DK)), v);
  };
  // indicators beyond the groups a thread holds in registers, and the last DK % 4
  auto put_ind_rest = [&](const float *irow) {
    for (int g = tl + TPE * NI; g < NG; g += TPE) put_ind(g, *reinterpret_cast<const env_f32x4u *>(irow + 4 * g));
    if (tl < (DK & 3)) {
      const float v = irow[4 * NG + tl] * d.s_ind;
      orow[1 + 2 * D + 4 * NG + tl] = v;
      O::store1(xrow(O::off(4 * NG + tl)), v);
    }
  };

  for (int i = tid; i < SE * XP / 4; i += kEnvThreads) reinterpret_cast<uint32_t *>(ldsX)[i] = 0u;
  __syncthreads();
  double value = 0.0;  // the account's, before the trades that are settled next
  float pn[1] = {a.price[((size_t)tau * d.M + (d.M == 1 ? 0 : n)) * D + dd]};
  if (trader) {
    if (own) put_holding(h[0]);
    if (live && tl == 0) put_cash(cash);
  }
  if (keeper) {
    const float *irow = a.ind + ((size_t)tau * d.M + (d.M == 1 ? 0 : n)) * DK;
    if (live) {
      for (int g = tl; g < min(NG, TPE * NI); g += TPE) put_ind(g, *reinterpret_cast<const env_f32x4u *>(irow + 4 * g));
      put_ind_rest(irow);
    }
    if (own) put_price(pn[0]);
    if (APART && tl < D) quote(pn[0], 0);
    terms_of(1);
    trade.put_term(0, tl < D ? (double)h[0] * (double)pn[0] : 0.0);
    value = trade.value(cash);
  }
  __syncthreads();

  const unsigned char *xop = ldsX + row * XP + O::off(8 * q4) + (SPLIT ? wt * B1 * 2 * O::KBYTES : 0);
  const unsigned char *h1op = ldsH1 + row * HP + O::off(8 * q4), *h2op = ldsH2 + row * HP + O::off(8 * q4);
  // tanh of this lane's sums into a hidden tile
  auto activate = [&](float (&z)[F], const float (&bias)[F], unsigned char *H) {
#pragma unroll
    for (int i = 0; i < F; ++i) {
      z[i] += bias[i];
      z[i] = BF16 ? tanh_from_scaled(z[i] * kTwoLog2e) : tanh_accurate(z[i]);
    }
    unsigned char *o = H + row * HP + O::off(f0);
    if constexpr (F == 4) O::template store4<true>(o, z[0], z[1], z[2], z[3]);
    else if constexpr (BF16) *reinterpret_cast<uint32_t *>(o) = bf16_pair(z[0], z[1]);
    else {
      uint32_t s[3];
      split3_pair<true>(z[0], z[1], s[0], s[1], s[2]);
#pragma unroll
      for (int i = 0; i < 3; ++i) *reinterpret_cast<uint32_t *>(o + 16 * i) = s[i];
    }
  };
  // a layer's products in two chains (one behind the other they wait for each other), and their sum
  auto product = [&](auto &wb, const unsigned char *x) {
    constexpr int NB = sizeof(wb) / sizeof(Block);
    Sums s[2];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      Block b;
      fetch_x(b, x + 2 * i * O::KBYTES);
      mma16(wb[i], b, s[i & 1].hi, s[i & 1].lo);
    }
    f32x4 v = NB > 1 ? s[0].hi + s[1].hi : s[0].hi;
    if (!BF16) v += NB > 1 ? s[0].lo + s[1].lo : s[0].lo;
    return v;
  };
  auto mine = [&](float (&z)[F], const f32x4 &v) {
#pragma unroll
    for (int i = 0; i < F; ++i) z[i] = F == 4 || wt == 0 ? v[i] : v[(2 + i) & 3];
  };
  // The books of step t (binary64; the first thread of an env holds the sums).  Nothing in the next step waits for them, so
  // wavefronts apart from the traders keep them while that step trades.
  auto settle = [&](int t, float c, bool ended) {
    terms_of(t);
    const double after = trade.value(c);
    const double r = (after - value) * (double)d.rho;
    value = ended ? (double)d.cash0 : after;
    ep_ret += r;
    if (ended) {
      ep_sum += ep_ret;
      ep_sqsum += ep_ret * ep_ret;
      ep_cnt += 1;
      ep_ret = 0.0;
    }
    if (live && tl == 0) {
      a.reward[(size_t)t * N + n] = (float)r;
      a.done[(size_t)t * N + n] = (uint8_t)ended;
    }
  };

  bool ended = false;
  for (int t = 0; t < a.T; ++t) {
    if (TIGHT) asm volatile("" : "+v"(tl), "+v"(e), "+v"(trade.me));
    const size_t g0 = ((size_t)t * N + n) * D;
    // -- requests of the step
    const RowInfo ri = rows_of(d, tau, start, n);
    float eps[1], pv[1], po;
    env_f32x4 iv[NI];
    const float *irow = a.ind + (size_t)ri.row_obs * DK;
    typename Tr::Unit units;
    if (trader) {
      eps[0] = __builtin_nontemporal_load(a.noise + g0 + dd);
      pv[0] = a.price[(size_t)ri.row_val * D + dd];
    }
    if (keeper) {
      po = a.price[(size_t)ri.row_obs * D + dd];
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const int g = tl + TPE * j;
        if (g < NG) iv[j] = *reinterpret_cast<const env_f32x4u *>(irow + 4 * g);
      }
    }
    if (!APART) units = Tr::unit_of(d, pn);
    // -- policy
    float f[F];
    {
      const f32x4 v = product(w1, xop);
      mine(f, v);
      if constexpr (SPLIT) {
        // the other wavefront's half of the k-steps for this one's features, and the other way round
        float other[F];
#pragma unroll
        for (int i = 0; i < F; ++i) other[i] = wt == 0 ? v[(2 + i) & 3] : v[i];
#pragma unroll
        for (int i = 0; i < F; ++i) share[(w * 2 + i) * kSharePitch + lane] = other[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < F; ++i) f[i] += share[((w ^ 4) * 2 + i) * kSharePitch + lane];
      }
    }
    activate(f, bias1, ldsH1);
    __syncthreads();
    mine(f, product(w2, h1op));
    activate(f, bias2, ldsH2);
    __syncthreads();
    if (ok < KS && 16 * ot < D) {
      Block w3s[1] = {w3};
      *reinterpret_cast<f32x4 *>(means + (ok * SE + row) * kMeanPitch + 16 * ot + 4 * q4) = product(w3s, h2op + 2 * ok * O::KBYTES);
    }
    __syncthreads();
    orow += N * S;
    // (layer 1 has read the present observation)
    auto move_market = [&]() {
      if (own) put_price(po);
      if (live) {
#pragma unroll
        for (int j = 0; j < NI; ++j) {
          const int g = tl + TPE * j;
          if (g < NG) put_ind(g, iv[j]);
        }
      }
    };
    if (trader) {
      // -- sample and trade
      if (APART) {
        __builtin_amdgcn_s_setprio(2);
        const Quote u = quotes[((t & 1) * SE + e) * QP + dd];
        pn[0] = u.price, units.cost[0] = u.cost, units.rcp[0] = u.rcp;
      }
      float z = 0.0f, a_raw[1];
#pragma unroll
      for (int k = 0; k < KS; ++k) z += means[(k * SE + e) * kMeanPitch + dd];
      const float mu = finish_out(z, bias3, 1);
      a_raw[0] = mu + d.sigma * eps[0];  // two roundings (contraction is off)
      if (own) {
        a.act_raw[g0 + tl] = a_raw[0];
        if (a.mu) a.mu[g0 + tl] = mu;
      }
      terms_of(t);
      int32_t q[1];
      float e2;
      double r;
      trade.run(
          d, live, a_raw, eps, pn, units, pv, h, q, cash, r, e2, a.logp != nullptr,
          [&]() {
            if (!APART) move_market();
          },
          [&]() {
            if (!APART && live) put_ind_rest(irow);
          },
          [&](int) {
            if (ri.done) h[0] = 0;
            put_holding(h[0]);
            if (a.shares) a.shares[g0 + tl] = q[0];
          });
      if (APART && tl == 0) balance[(t & 1) * SE + e] = cash;
      if (!APART) settle(t, cash, ri.done);
      if (ri.done) cash = d.cash0;
      if (live && tl == 0) {
        put_cash(cash);
        if (a.logp) a.logp[(size_t)t * N + n] = fmaf(-0.5f, e2, d.logp_const);
      }
      if (APART) __builtin_amdgcn_s_setprio(0);
      else pn[0] = po;
    } else {
      move_market();
      if (tl < D) quote(po, (t + 1) & 1);
      if (live) put_ind_rest(irow);
      if (t > 0) settle(t - 1, balance[((t - 1) & 1) * SE + e], ended);
      ended = ri.done;
    }
    tau = ri.done ? start : tau + 1;
    __syncthreads();  // the next observation is complete
  }

  if (trader) {
    if (own) a.st.h[(size_t)n * D + tl] = h[0];
    if (live && tl == 0) a.st.tau[n] = tau, a.st.cash[n] = cash;
  }
  if (keeper) {
    if (APART && a.T > 0) settle(a.T - 1, balance[((a.T - 1) & 1) * SE + e], ended);
    if (live && tl == 0) {
      a.st.ep_ret[n] = ep_ret;
      a.st.ep_sum[n] = ep_sum;
      a.st.ep_sqsum[n] = ep_sqsum;
      a.st.ep_cnt[n] = ep_cnt;
    }
  }
}

template <bool BF16, int HD, int KS1, bool SPLIT, bool APART>
hipError_t launch_stocks(hipStream_t st, const SmallArgs &a) {
  constexpr int KS = Geometry<HD>::KS;
  constexpr auto kern = rollout_small_kernel<BF16, HD, KS1, SPLIT, APART>;
  const hipError_t e = allow_full_lds<kern>();
  if (e != hipSuccess) return e;
  const size_t lds = small_lds(KS, SPLIT, APART, tile::tile_pitch<BF16>(2 * KS1), tile::tile_pitch<BF16>(2 * KS), a.d.D);
  hipLaunchKernelGGL(kern, dim3((unsigned)((a.d.N + SE - 1) / SE)), dim3(kEnvThreads), lds, st, a);
  return hipGetLastError();
}

template <bool BF16, int HD, int KS1, bool SPLIT = false>
hipError_t launch_inst(hipStream_t st, const SmallArgs &a) {
  return a.d.D <= 16 ? launch_stocks<BF16, HD, KS1, SPLIT, true>(st, a) : launch_stocks<BF16, HD, KS1, SPLIT, false>(st, a);
}

template <bool BF16>
hipError_t launch_dtype(hipStream_t st, const SmallArgs &a) {
  const int nkb = a.net.nkb[0];
  // the smallest instance whose wavefronts hold layer 1: inputs beyond the last are multiplied by zeros
  if (a.net.nct[0] == 2) {
    if (nkb <= 2) return launch_inst<BF16, 64, 1>(st, a);
    if (nkb <= 4) return launch_inst<BF16, 64, 2>(st, a);
    if (nkb <= 8) return launch_inst<BF16, 64, 4, !BF16>(st, a);
    return launch_inst<BF16, 64, 10, !BF16>(st, a);
  }
  if (nkb <= 4) return launch_inst<BF16, 128, 2>(st, a);
  if (nkb <= 10) return launch_inst<BF16, 128, 5>(st, a);
  return launch_inst<BF16, 128, 10>(st, a);
}

// ---------------------------------------------------------------- value head
struct ValueSmallArgs {
  const float *X;   // [rows][S]
  int64_t rows;
  PackedNet net;
  int32_t S, N, envs_per_agent, per_agent;  // per_agent: workgroups of an agent
  float *Y;
};

// The critic of such a rollout over its record: eight wavefronts own 16 features each of 16 rows (128 hidden units) or 32, with the
// weights in registers from the first tile to the last.  A tile's rows are requested behind the products of the one before;
// the output layer's one feature is summed from the activations where they are formed.
// Bound by the products, 16 x 16 x 32 instructions, where there are many rows and by two barriers and the rows' round trip
// where there are few.  The kernels for any network it takes the place of kept a tile's weights in a ring and a last
// tile that is not full had a launch of its own (9 us).  Rollouts with values, fp32: 512 envs x 30 stocks x 8, 64 units, 64 steps
// 341 -> 315 us, 16384, 32 steps 1230 -> 945; 4096 with 128 units 471 -> 418, 300 x 12 x 4 261 -> 242; bf16, 333 x 17 x 5 198 -> 177.
template <bool BF16, int HD, int KS1>
__global__ __launch_bounds__(kEnvThreads, 2) void value_small_kernel(ValueSmallArgs a) {
  using namespace tile;
  using O = Op<BF16>;
  using Block = typename O::Block;
  constexpr int TILES = HD / 16, RT = kWaves / TILES, RR = 16 * RT, TPR = kEnvThreads / RR, KS = HD / 32, NCT = HD / 32;
  constexpr int NP = 64 * kPlanes<Block>, GROUPS = (8 * KS1 + TPR - 1) / TPR;
  constexpr int XP = tile_pitch<BF16>(2 * KS1), HP = tile_pitch<BF16>(2 * KS);
  __shared__ __align__(16) unsigned char ldsX[RR * XP];
  __shared__ __align__(16) unsigned char ldsH[RR * HP];
  __shared__ float part[TILES * RR];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ft = w % TILES, rt = w / TILES, q4 = lane >> 4, row = lane & 15, S = a.S;

  // tiles of an agent: its rows in each step; of a single one the rows as they are
  const bool several = a.envs_per_agent < a.N;
  const int block = (int)(several ? xcd_run(blockIdx.x, gridDim.x) : blockIdx.x), agent = block / a.per_agent, first = block - agent * a.per_agent;
  const int64_t in_step = several ? a.envs_per_agent / RR : 1;
  const int64_t tiles = several ? a.rows / a.N * in_step : (a.rows + RR - 1) / RR;
  auto row0_of = [&](int64_t k) {
    if (!several) return k * RR;
    const int64_t t = k / in_step;
    return t * a.N + (int64_t)agent * a.envs_per_agent + (k - t * in_step) * RR;
  };

  const Net net = net_of(a.net, agent);
  auto fetch = [&](Block &b, const u32x4 *W, int nkb, int ks) {
    const int kb = 2 * ks + (q4 >> 1);
    if constexpr (!BF16 || skips_blocks(BF16, HD, KS1)) {  // (few registers are held here)
      b = Block{};
      if (kb < nkb) fetch_w(b, W + ((size_t)kb * NCT + (ft >> 1)) * NP + (ft & 1) * 16 + row + 32 * (q4 & 1));
    } else {
      fetch_w(b, W + ((size_t)min(kb, nkb - 1) * NCT + (ft >> 1)) * NP + (ft & 1) * 16 + row + 32 * (q4 & 1));
      if (kb >= nkb) b = Block{};
    }
  };
  Block w1[KS1], w2[KS];
#pragma unroll
  for (int i = 0; i < KS1; ++i) fetch(w1[i], net.W[0], net.nkb[0], i);
#pragma unroll
  for (int i = 0; i < KS; ++i) fetch(w2[i], net.W[1], 2 * KS, i);
  const int f0 = 16 * ft + 4 * q4;
  const f32x4 bias1 = *reinterpret_cast<const f32x4 *>(net.b[0] + f0), bias2 = *reinterpret_cast<const f32x4 *>(net.b[1] + f0);
  f32x4 w3;  // (feature 0 of the packed output layer: input 16 kb + 8 g + e sits in lane 32 g)
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int f = f0 + i;
    const __bf16 *p = reinterpret_cast<const __bf16 *>(net.W[2] + (size_t)(f >> 4) * NP + 32 * ((f >> 3) & 1)) + (f & 7);
    w3[i] = (float)p[0];
    if (!BF16) w3[i] = w3[i] + ((float)p[512] + (float)p[1024]);
  }
  const float b3 = net.b[2][0];

  for (int i = tid; i < RR * XP / 4; i += kEnvThreads) reinterpret_cast<uint32_t *>(ldsX)[i] = 0u;
  const int e = tid / TPR, tl = tid & (TPR - 1);
  f32x4 pre[GROUPS];
  auto request = [&](int64_t k) {
    const float *x = a.X + min(row0_of(min(k, tiles - 1)) + e, a.rows - 1) * S;
#pragma unroll
    for (int g = 0; g < GROUPS; ++g) {
      const int c = 4 * (tl + TPR * g);
      if (c + 4 <= S) pre[g] = *reinterpret_cast<const env_f32x4u *>(x + c);
      else if (c < S) pre[g] = f32x4{x[c], c + 1 < S ? x[c + 1] : 0.0f, c + 2 < S ? x[c + 2] : 0.0f, 0.0f};
    }
  };
  auto stash = [&]() {
#pragma unroll
    for (int g = 0; g < GROUPS; ++g) {
      const int c = 4 * (tl + TPR * g);
      if (c < S) O::store4(ldsX + e * XP + O::off(c), pre[g][0], pre[g][1], pre[g][2], pre[g][3]);
    }
  };
  const unsigned char *xop = ldsX + (16 * rt + row) * XP + O::off(8 * q4), *hop = ldsH + (16 * rt + row) * HP + O::off(8 * q4);
  auto product = [&](auto &wb, const unsigned char *x, const f32x4 &bias) {
    constexpr int NB = sizeof(wb) / sizeof(Block);
    Sums s[2];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      Block b;
      fetch_x(b, x + 2 * i * O::KBYTES);
      mma16(wb[i], b, s[i & 1].hi, s[i & 1].lo);
    }
    f32x4 v = s[0].hi + s[1].hi;
    if (!BF16) v += s[0].lo + s[1].lo;
    v += bias;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = BF16 ? tanh_from_scaled(v[i] * kTwoLog2e) : tanh_accurate(v[i]);
    return v;
  };
  auto finish = [&](int64_t k) {
    if (tid < RR) {
      float y = b3;
#pragma unroll
      for (int i = 0; i < TILES; ++i) y += part[i * RR + tid];
      const int64_t r = row0_of(k) + tid;
      if (r < a.rows) a.Y[r] = y;
    }
  };

  if (first >= tiles) return;
  request(first);
  __syncthreads();  // (the zeros)
  stash();
  for (int64_t k = first; k < tiles; k += a.per_agent) {
    __syncthreads();  // the tile's rows, and the sums of the one before
    if (k > first) finish(k - a.per_agent);
    request(k + a.per_agent);
    const f32x4 h1 = product(w1, xop, bias1);
    O::template store4<true>(ldsH + (16 * rt + row) * HP + O::off(f0), h1[0], h1[1], h1[2], h1[3]);
    __syncthreads();
    const f32x4 h2 = product(w2, hop, bias2);
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) s = fmaf(BF16 ? (float)(__bf16)h2[i] : h2[i], w3[i], s);
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 32);
    if (q4 == 0) part[ft * RR + 16 * rt + row] = s;
    stash();
  }
  __syncthreads();
  finish(first + (tiles - 1 - first) / a.per_agent * a.per_agent);
}

template <bool BF16, int HD, int KS1>
hipError_t launch_value_inst(hipStream_t st, ValueSmallArgs a, int cus) {
  constexpr int RR = 16 * (kWaves / (HD / 16));
  const int agents = a.N / a.envs_per_agent;
  const int64_t tiles = agents > 1 ? a.rows / a.N * (a.envs_per_agent / RR) : (a.rows + RR - 1) / RR;
  a.per_agent = (int32_t)std::min<int64_t>(tiles, std::max(1, cus / agents));
  hipLaunchKernelGGL((value_small_kernel<BF16, HD, KS1>), dim3((unsigned)(a.per_agent * agents)), dim3(kEnvThreads), 0, st, a);
  return hipGetLastError();
}

template <bool BF16>
hipError_t launch_value_dtype(hipStream_t st, const ValueSmallArgs &a, int cus) {
  const int nkb = a.net.nkb[0];
  if (a.net.nct[0] == 2) {
    if (nkb <= 2) return launch_value_inst<BF16, 64, 1>(st, a, cus);
    if (nkb <= 4) return launch_value_inst<BF16, 64, 2>(st, a, cus);
    if (nkb <= 8) return launch_value_inst<BF16, 64, 4>(st, a, cus);
    return launch_value_inst<BF16, 64, 10>(st, a, cus);
  }
  if (nkb <= 4) return launch_value_inst<BF16, 128, 2>(st, a, cus);
  if (nkb <= 10) return launch_value_inst<BF16, 128, 5>(st, a, cus);
  return launch_value_inst<BF16, 128, 10>(st, a, cus);
}

}  // namespace

// 64 or 128 hidden units, up to 320 inputs and 32 stocks: what eight wavefronts hold in registers.
// A round of workgroups, one per compute unit, is 4096 envs, and the launches per step that would take over (query_kernel or
// mlp_tiles_kernel, and an env step) win only for calls of a step or a few of very many envs in fp32 with 128 units on more than 160 inputs,
// where the start of a workgroup costs more than a step: 65536 envs x 30, one step 365 -> 508 us, two 298 -> 353 a step, four 264
// -> 272, eight 246 -> 232, sixteen 236 -> 212; 16384 envs of 16 agents, one 114 -> 128, two 92 -> 86.  (All calls take the one launch:
// a rollout gives the same bits however it is cut into calls.)  Rollouts with values of 24 steps, 16 of 16384 envs and 6 of 65536; us, this and those:
//   envs                         512           4096          8192          16384          65536
//   fp32, 128 units, 301     203 and 359   324 and 525   639 and 903   871 and 1166  1498 and 1629
//   fp32, 128 units, 151     109 and 328   181 and 438   327 and 694   446 and 854    792 and 1204
//   fp32,  64 units, 301     132 and 344   191 and 470   372 and 793   505 and 1025   876 and 1420
//   bf16, 128 units, 301      97 and 292   150 and 345   310 and 500   429 and 726    738 and 808
bool small_supported(const pr_config &c) {
  const int S = 1 + 2 * c.n_stocks + c.n_stocks * c.n_ind;
  return c.schedule == PR_SCHED_STEPWISE && (c.hidden == 64 || c.hidden == 128) && c.n_stocks <= 32 && S <= 16 * kMaxBlocks;
}

hipError_t launch_rollout_small(hipStream_t st, const EnvDims &d, const EnvState &s, const float *price, const float *ind,
                                const PackedNet &actor, int32_t envs_per_agent, int32_t T, const float *noise,
                                const pr_buffers &out) {
  SmallArgs a;
  a.d = d, a.st = s, a.price = price, a.ind = ind, a.net = actor, a.envs_per_agent = envs_per_agent, a.T = T, a.noise = noise;
  a.obs = out.obs, a.act_raw = out.act_raw, a.reward = out.reward, a.done = out.done, a.logp = out.logp, a.mu = out.mu;
  a.shares = out.shares;
  // An agent's workgroups on one XCD, which then has its weights from memory once: fp32, 64 units, 301 inputs, us a call of one step
  // with values, 64 agents of 64 envs 37.5 -> 27.7, 8 agents of 64 25.6 -> 24.0; bf16 21.5 -> 16.2.  One agent's envs of any number are
  // slower in runs (65536 x 30 in bf16 187 -> 198), and so are many envs of bf16 networks, whose weights are few (64 agents 196 -> 201).
  a.runs = envs_per_agent < d.N && (!actor.bf16 || d.N <= 1024 * SE);
  return actor.bf16 ? launch_dtype<true>(st, a) : launch_dtype<false>(st, a);
}

// Where other kernels of the forward pass are the faster value head.  Up to 4096 rows of more than 64 inputs: query_kernel, which starts
// on the rows at once; us of the head behind calls of four steps, this -> that: fp32, 64 units, 301 inputs, 5 rows 9.1 -> 6.2, 500 10.9 -> 6.9,
// 4000 11.7 -> 8.5; 73 inputs 2000 rows 6.6 -> 6.0; bf16, 128 units, 301 inputs 500 rows 5.7 -> 4.5; up to 64 inputs level or the other way
// round.  Many rows in bf16 of more than 160 inputs, which pay for 320 here: 128 units, 301 inputs, 20480 rows 9.8 -> 8.7 the
// other way round, 30000 14.2 -> 14.0, 81920 29.3 -> 27.8, 327680 131 -> 115 (161 inputs 101 -> 88), 64 units 163840 level, 327680 111 -> 108.
bool value_small_covers(const PackedNet &critic, int64_t rows) {
  const int nkb = critic.nkb[0], hidden = critic.out_dim[0];
  if (nkb > 4 && rows <= 4096) return false;
  return !(critic.bf16 && nkb > 10 && rows > (hidden == 64 ? 200000 : 24576));
}

hipError_t launch_value_small(hipStream_t st, const PackedNet &critic, int64_t rows, const float *X, int32_t S, float *Y, int32_t N,
                              int32_t envs_per_agent, int cus) {
  ValueSmallArgs a;
  a.X = X, a.rows = rows, a.net = critic, a.S = S, a.N = N, a.envs_per_agent = envs_per_agent, a.per_agent = 1, a.Y = Y;
  return critic.bf16 ? launch_value_dtype<true>(st, a, cus) : launch_value_dtype<false>(st, a, cus);
}

}  // namespace pod
