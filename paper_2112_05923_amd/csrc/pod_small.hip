// The stepwise schedule's rollout for small networks: one launch for all T steps.
//
// With 64 or 128 hidden units a step is a few microseconds of launches around a
// few hundred nanoseconds of work: 17 us for 16 envs, whatever the device does.
// Envs are independent, so a workgroup keeps 16 of them, their state and the
// WHOLE policy network on its compute unit instead: the weights stay in registers
// from the first step to the last, the observation lives in LDS as the operand
// layer 1 reads, and only the rollout's records go to memory.
//
// What bounds a step is latency: three layers of one to ten matrix steps per
// wavefront, each followed by two barriers (partial sums, activations), then the
// trades' chain (pod_trade.h).  The loads of a step -- noise, the next market row
// -- depend on the cursor only and travel behind the network.
// Per step, before (a network launch or three and an env launch) -> now:
//   fp32,  64 hidden units: 16 envs x 5 stocks 19.6 -> 3.6 us, 512 x 30 x 8 indicators 30 -> 5.1, 16384 x 30 x 8 55 -> 21
//   fp32, 128: 64 x 10 x 2 27 -> 5.5, 512 x 30 x 8 37 -> 10.9 (129 of its registers spill; 28 with up to 160 inputs),
//   4096 x 30 x 8 40 -> 15
//   bf16, 128: 512 x 30 x 8 30 -> 4.2, 16384 x 30 x 8 38 -> 18
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
  const float *noise;  // [T, N, D]
  float *obs;          // [T+1, N, S]
  float *act_raw;      // [T, N, D]
  float *reward;       // [T, N]
  uint8_t *done;       // [T, N]
  float *logp;         // opt [T, N]
  float *mu;           // opt [T, N, D]
  int32_t *shares;     // opt [T, N, D]
};

template <int NCT>
struct Geometry {
  static constexpr int HD = 32 * NCT;          // hidden units
  static constexpr int KG = kWaves / NCT;      // wavefronts that share a feature tile's k-blocks
  static constexpr int F = HD * SE / kEnvThreads;  // features per thread between the layers
  static constexpr int PP = HD + 4;            // row pitch of a plane of partial sums
  static constexpr int NKB = HD / 16;          // k-blocks of layers 2 and 3
};

// NCT: hidden feature tiles (2 or 4); B1: layer-1 k-blocks per wavefront
template <bool BF16, int NCT, int B1>
__global__ __launch_bounds__(kEnvThreads, 2) void rollout_small_kernel(SmallArgs a) {
  using namespace tile;
  using O = Op<BF16>;
  using Block = typename O::Block;
  using Gm = Geometry<NCT>;
  using Tr = Trade<SE, 1, true>;
  constexpr int TPE = Tr::TPE, NI = 4, KG = Gm::KG, F = Gm::F, B2 = Gm::NKB / KG;
  constexpr int XP = tile_pitch<BF16>(B1 * KG), HP = tile_pitch<BF16>(Gm::NKB);
  extern __shared__ __align__(16) unsigned char lds[];
  const EnvDims &d = a.d;
  const int D = d.D, DK = D * d.K, S = d.S, NG = DK / 4;
  unsigned char *ldsX = lds, *ldsH = ldsX + SE * XP;
  float *part = reinterpret_cast<float *>(ldsH + SE * HP);  // [KG][SE][PP], and [NKB][SE][36] for the output layer
  unsigned char *ldsT = reinterpret_cast<unsigned char *>(part + (KG * Gm::PP > Gm::NKB * 36 ? KG * Gm::PP : Gm::NKB * 36) * SE);
  Tr trade(ldsT, D);

  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int e = tid / TPE, tl = tid & (TPE - 1), dd = min(tl, D - 1);
  const int n0 = blockIdx.x * SE, n = min(n0 + e, d.N - 1);
  const bool live = n0 + e < d.N, own = live && tl < D;
  const size_t N = (size_t)d.N;

  // -- the network: this wavefront's weight blocks, this thread's biases
  const Net net = net_of(a.net, (n0 % d.N) / a.envs_per_agent);
  const int ct = w % NCT, kg = w / NCT;
  Block w1[B1], w2[B2], w3;
#pragma unroll
  for (int i = 0; i < B1; ++i) {
    const int kb = kg + KG * i;
    w1[i] = Block{};
    if (kb < net.nkb[0]) fetch_w(w1[i], net.W[0] + ((size_t)kb * NCT + ct) * (64 * kPlanes<Block>) + lane);
  }
  // (fp32 with 128 hidden units: layer 2's blocks would not fit next to the others and are read again in every step)
  constexpr bool KEEP2 = BF16 || NCT == 2;
  auto fetch2 = [&](int lane_f) {
#pragma unroll
    for (int i = 0; i < B2; ++i) fetch_w(w2[i], net.W[1] + ((size_t)(kg + KG * i) * NCT + ct) * (64 * kPlanes<Block>) + lane_f);
  };
  if (KEEP2) fetch2(lane);
  fetch_w(w3, net.W[2] + (size_t)min(w, Gm::NKB - 1) * (64 * kPlanes<Block>) + lane);
  const int f0 = tl * F;  // this thread's features of row e, between the layers
  float bias1[F], bias2[F];
#pragma unroll
  for (int i = 0; i < F; ++i) bias1[i] = net.b[0][f0 + i], bias2[i] = net.b[1][f0 + i];
  const float bias3 = net.b[2][tl];

  // -- state
  int32_t tau = a.st.tau[n];
  const int32_t start = a.st.start[n];
  float cash = a.st.cash[n];
  int32_t h[1] = {a.st.h[(size_t)n * D + dd]};
  double ep_ret = a.st.ep_ret[n], ep_sum = a.st.ep_sum[n], ep_sqsum = a.st.ep_sqsum[n];
  int32_t ep_cnt = a.st.ep_cnt[n];

  unsigned char *xrow = ldsX + e * XP;
  float *orow = a.obs + (size_t)n * S;  // of the observation being written
  auto put_ind = [&](int g, env_f32x4 v) {
    v[0] *= d.s_ind, v[1] *= d.s_ind, v[2] *= d.s_ind, v[3] *= d.s_ind;
    *reinterpret_cast<env_f32x4u *>(orow + 1 + 2 * D + 4 * g) = v;
    O::store4(xrow + O::off(4 * g), v[0], v[1], v[2], v[3]);
  };
  auto put_price = [&](float p) {
    const float v = p * d.s_price;
    orow[1 + tl] = v;
    O::store1(xrow + O::off(DK + 1 + tl), v);
  };
  auto put_holding = [&](int32_t x) {
    const float v = (float)x * d.s_hold;
    orow[1 + D + tl] = v;
    O::store1(xrow + O::off(DK + 1 + D + tl), v);
  };
  auto put_cash = [&](float c) {
    const float v = c * d.s_cash;
    orow[0] = v;
    O::store1(xrow + O::off(DK), v);
  };
  // indicators beyond the groups a thread holds in registers, and the last DK % 4
  auto put_ind_rest = [&](const float *irow) {
    for (int g = tl + TPE * NI; g < NG; g += TPE) put_ind(g, *reinterpret_cast<const env_f32x4u *>(irow + 4 * g));
    if (tl < (DK & 3)) {
      const float v = irow[4 * NG + tl] * d.s_ind;
      orow[1 + 2 * D + 4 * NG + tl] = v;
      O::store1(xrow + O::off(4 * NG + tl), v);
    }
  };

  for (int i = tid; i < SE * XP / 4; i += kEnvThreads) reinterpret_cast<uint32_t *>(ldsX)[i] = 0u;
  __syncthreads();
  float pn[1];
  {
    const size_t row = (size_t)tau * d.M + (d.M == 1 ? 0 : n);
    const float *irow = a.ind + row * DK;
    pn[0] = a.price[row * D + dd];
    if (live) {
      for (int g = tl; g < min(NG, TPE * NI); g += TPE) put_ind(g, *reinterpret_cast<const env_f32x4u *>(irow + 4 * g));
      put_ind_rest(irow);
      if (tl == 0) put_cash(cash);
    }
    if (own) put_price(pn[0]), put_holding(h[0]);
  }
  trade.put_term(0, tl < D ? (double)h[0] * (double)pn[0] : 0.0);
  double value = trade.value(cash);  // the account's, before the next trades
  __syncthreads();

  // partial sums of feature tile `tile`, lanes of the 16 rows only
  const unsigned char *xop = ldsX + (lane & 15) * XP + O::HALF * (lane >> 5);
  const unsigned char *hop = ldsH + (lane & 15) * HP + O::HALF * (lane >> 5);
  auto put_part = [&](const f32x16 &acc, float *plane, int pitch, int col0) {
    if ((lane & 31) < SE) {
      float *p = plane + (lane & 15) * pitch + col0 + 4 * (lane >> 5);
#pragma unroll
      for (int j = 0; j < 4; ++j) *reinterpret_cast<f32x4 *>(p + 8 * j) = f32x4{acc[4 * j], acc[4 * j + 1], acc[4 * j + 2], acc[4 * j + 3]};
    }
  };
  // hidden activations of this thread's features from the partial sums
  auto activate = [&](const float (&bias)[F]) {
    float z[F];
#pragma unroll
    for (int i = 0; i < F; ++i) z[i] = bias[i];
#pragma unroll
    for (int k = 0; k < KG; ++k) {
      const float *p = part + (k * SE + e) * Gm::PP + f0;
#pragma unroll
      for (int i = 0; i < F; ++i) z[i] += p[i];
    }
#pragma unroll
    for (int i = 0; i < F; ++i) z[i] = BF16 ? tanh_from_scaled(z[i] * kTwoLog2e) : tanh_accurate(z[i]);
    unsigned char *o = ldsH + e * HP + O::off(f0);
    if constexpr (F == 4) O::template store4<true>(o, z[0], z[1], z[2], z[3]);
    else if constexpr (BF16) *reinterpret_cast<uint32_t *>(o) = bf16_pair(z[0], z[1]);
    else {
      uint32_t s[3];
      split3_pair<true>(z[0], z[1], s[0], s[1], s[2]);
#pragma unroll
      for (int i = 0; i < 3; ++i) *reinterpret_cast<uint32_t *>(o + 16 * i) = s[i];
    }
  };
  auto zero = [](f32x16 &acc) {
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
  };

  for (int t = 0; t < a.T; ++t) {
    const size_t g0 = ((size_t)t * N + n) * D;
    // -- requests of the step
    if (!KEEP2) {
      int lane_f = lane;
      asm volatile("" : "+v"(lane_f));
      fetch2(lane_f);
    }
    const RowInfo ri = rows_of(d, tau, start, n);
    float eps[1], pv[1];
    eps[0] = __builtin_nontemporal_load(a.noise + g0 + dd);
    pv[0] = a.price[(size_t)ri.row_val * D + dd];
    const float po = a.price[(size_t)ri.row_obs * D + dd];
    const float *irow = a.ind + (size_t)ri.row_obs * DK;
    env_f32x4 iv[NI];
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int g = tl + TPE * j;
      if (g < NG) iv[j] = *reinterpret_cast<const env_f32x4u *>(irow + 4 * g);
    }
    const typename Tr::Unit units = Tr::unit_of(d, pn);
    // -- policy
    f32x16 acc;
    zero(acc);
#pragma unroll
    for (int i = 0; i < B1; ++i) {
      Block x;
      fetch_x(x, xop + (kg + KG * i) * O::KBYTES);
      O::mma(w1[i], x, acc);
    }
    put_part(acc, part + kg * SE * Gm::PP, Gm::PP, ct * 32);
    __syncthreads();
    activate(bias1);
    __syncthreads();
    zero(acc);
#pragma unroll
    for (int i = 0; i < B2; ++i) {
      Block x;
      fetch_x(x, hop + (kg + KG * i) * O::KBYTES);
      O::mma(w2[i], x, acc);
    }
    put_part(acc, part + kg * SE * Gm::PP, Gm::PP, ct * 32);
    __syncthreads();
    activate(bias2);
    __syncthreads();
    if (w < Gm::NKB) {
      zero(acc);
      Block x;
      fetch_x(x, hop + w * O::KBYTES);
      O::mma(w3, x, acc);
      put_part(acc, part + w * SE * 36, 36, 0);
    }
    __syncthreads();
    float z = 0.0f;
#pragma unroll
    for (int k = 0; k < Gm::NKB; ++k) z += part[(k * SE + e) * 36 + tl];
    const float mu = finish_out(z, bias3, 1);
    // -- sample and trade
    float a_raw[1];
    a_raw[0] = mu + d.sigma * eps[0];  // two roundings (contraction is off)
    if (own) {
      a.act_raw[g0 + tl] = a_raw[0];
      if (a.mu) a.mu[g0 + tl] = mu;
    }
    orow += N * S;
    int32_t q[1];
    float e2;
    double r;
    trade.run(
        d, live, a_raw, eps, pn, units, pv, h, q, cash, r, e2, a.logp != nullptr,
        [&]() {
          if (own) put_price(po);
          if (live) {
#pragma unroll
            for (int j = 0; j < NI; ++j) {
              const int g = tl + TPE * j;
              if (g < NG) put_ind(g, iv[j]);
            }
          }
        },
        [&]() {
          if (live) put_ind_rest(irow);
        },
        [&](int) {
          if (ri.done) h[0] = 0;
          put_holding(h[0]);
          if (a.shares) a.shares[g0 + tl] = q[0];
        });
    // -- episode bookkeeping (binary64; the env's first thread holds the sums), reset if the episode ended
    const double after = trade.value(cash);
    r = (after - value) * (double)d.rho;
    value = ri.done ? (double)d.cash0 : after;
    ep_ret += r;
    if (ri.done) {
      ep_sum += ep_ret;
      ep_sqsum += ep_ret * ep_ret;
      ep_cnt += 1;
      ep_ret = 0.0;
      cash = d.cash0;
    }
    tau = ri.done ? start : tau + 1;
    pn[0] = po;
    if (live && tl == 0) {
      put_cash(cash);
      a.reward[(size_t)t * N + n] = (float)r;
      a.done[(size_t)t * N + n] = (uint8_t)ri.done;
      if (a.logp) a.logp[(size_t)t * N + n] = fmaf(-0.5f, e2, d.logp_const);
    }
    __syncthreads();  // the next observation is complete
  }

  if (own) a.st.h[(size_t)n * D + tl] = h[0];
  if (live && tl == 0) {
    a.st.tau[n] = tau;
    a.st.cash[n] = cash;
    a.st.ep_ret[n] = ep_ret;
    a.st.ep_sum[n] = ep_sum;
    a.st.ep_sqsum[n] = ep_sqsum;
    a.st.ep_cnt[n] = ep_cnt;
  }
}

template <bool BF16, int NCT, int B1>
hipError_t launch_inst(hipStream_t st, const SmallArgs &a) {
  using Gm = Geometry<NCT>;
  constexpr auto kern = rollout_small_kernel<BF16, NCT, B1>;
  const hipError_t e = allow_full_lds<kern>();
  if (e != hipSuccess) return e;
  const size_t planes = Gm::KG * Gm::PP > Gm::NKB * 36 ? Gm::KG * Gm::PP : Gm::NKB * 36;
  const size_t lds = (size_t)SE * (tile::tile_pitch<BF16>(B1 * Gm::KG) + tile::tile_pitch<BF16>(Gm::NKB)) + planes * SE * 4 +
                     trade_lds(SE, true, a.d.D);
  hipLaunchKernelGGL(kern, dim3((unsigned)((a.d.N + SE - 1) / SE)), dim3(kEnvThreads), lds, st, a);
  return hipGetLastError();
}

template <bool BF16>
hipError_t launch_dtype(hipStream_t st, const SmallArgs &a) {
  const int nkb = a.net.nkb[0];
  // the smallest instance whose wavefronts hold layer 1: blocks beyond the last are multiplied by zeros
  if (a.net.nct[0] == 2) {
    if (nkb <= 4) return launch_inst<BF16, 2, 1>(st, a);
    if (nkb <= 8) return launch_inst<BF16, 2, 2>(st, a);
    return launch_inst<BF16, 2, 5>(st, a);
  }
  if (nkb <= 4) return launch_inst<BF16, 4, 2>(st, a);
  if (nkb <= 10) return launch_inst<BF16, 4, 5>(st, a);
  return launch_inst<BF16, 4, 10>(st, a);
}

}  // namespace

// 64 or 128 hidden units, up to 320 inputs and 32 stocks: what eight wavefronts hold in registers.
// A round of workgroups, one per compute unit, is 4096 envs.  The launches per step that take over cost about 17 us and
// then grow more slowly, so the line lies where they win over a rollout of 24 steps; us per step, this kernel and those:
//   fp32, 128 units, 301 inputs (129 registers spill): 4096 envs 15.1 and 21.7, 8192 30.5 and 34.9, 12288 45.7 and 42.7,
//   65536 241 and 152; 171 inputs: 8192 29.0 and 29.3, 12288 43.5 and 34.1
//   fp32, 128 units, 151 inputs: 4096 6.6 and 19.1, 65536 104 and 116; 61 inputs: 65536 97 and 103
//   fp32, 64 units, 301 inputs: 4096 5.4 and 18.0, 65536 83 and 136; bf16, 128 units, 301 inputs: 65536 71 and 86
// The state and the policy are loaded once a call, so a call of a single step has less of it (us): fp32, 128 units, 301 inputs
// 4096 envs 35 and 30, 8192 63 and 43; 151 inputs 4096 18 and 25, 16384 52 and 45, 65536 193 and 139; bf16 301 inputs
// 4096 13 and 26, 65536 151 and 138.  The number of steps is not asked: a rollout gives the same bits however it is cut.
bool small_supported(const pr_config &c) {
  const int S = 1 + 2 * c.n_stocks + c.n_stocks * c.n_ind;
  if (c.mlp_dtype == PR_MLP_F32 && c.hidden == 128 && S > 160 && c.n_envs > 8192) return false;
  return c.schedule == PR_SCHED_STEPWISE && (c.hidden == 64 || c.hidden == 128) && c.n_stocks <= 32 && S <= 16 * kMaxBlocks;
}

hipError_t launch_rollout_small(hipStream_t st, const EnvDims &d, const EnvState &s, const float *price, const float *ind,
                                const PackedNet &actor, int32_t envs_per_agent, int32_t T, const float *noise,
                                const pr_buffers &out) {
  SmallArgs a;
  a.d = d, a.st = s, a.price = price, a.ind = ind, a.net = actor, a.envs_per_agent = envs_per_agent, a.T = T, a.noise = noise;
  a.obs = out.obs, a.act_raw = out.act_raw, a.reward = out.reward, a.done = out.done, a.logp = out.logp, a.mu = out.mu;
  a.shares = out.shares;
  return actor.bf16 ? launch_dtype<true>(st, a) : launch_dtype<false>(st, a);
}

}  // namespace pod
