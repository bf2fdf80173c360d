// Persistent rollout kernel for fp32 networks of 256 hidden units: one workgroup keeps
// 16 or 32 envs on its compute unit for all T steps (the worker of Sec. 4.2; see
// pod_fused.hip, which has the bf16 networks).
//
// A step is a chain -- observation, three layers, sample, trade, observation.  Four
// wavefronts run the network, a SIMD each, four others the envs, and what depends on no
// decision leaves the chain:
//   network                                   envs (sixteen or eight threads each)
//   layer 1, the portfolio's columns, tanh    reward of step t - 1; request noise and the next market rows
//   --- hidden layer complete, input free
//   layer 2, tanh, output layer               write the market rows of observation t + 1 (records and input tile)
//   --- means complete, hidden tile free
//   layer 1 of step t + 1, market columns     sample, size, trade (pod_trade.h), portfolio columns
//   --- observation t + 1 complete
// The two kinds of wavefront run separate loops with the same barriers: neither's
// registers are live in the other's code.
//
// Bound with 16 envs by the weight stream -- 800 KB a step, which a compute unit takes in
// at 64 B a clock, 6.6 us at the 1.9 GHz this runs at; 84 KB of layer 2 stay in LDS and the
// output layer's 48 KB in registers (without either 12.3 us a step for 11.4) -- and by the
// chains beside it: two epilogues of 1 us, trades 3 us; the matrix pipe is busy 38 % of a
// step.  With 32 envs the matrix instructions take as long as the stream: 8 us of 17.6, the
// chip at 1.75-1.8 GHz (counters of both: profiles/pmc_fp32_kernels.txt).
// 301 inputs, per step, against 32 envs whose eight wavefronts all take turns at network
// and envs: 1024 envs 16.2 -> 8.2 us, 4096 16.9 -> 10.9, 8192 20.4 -> 17.2, 16384 37.9 ->
// 34.0, 65536 of 64 agents 151 -> 135; 12 stocks x 4 indicators, 4096 envs, 14.2 -> 8.4.
//
// Compiled with floating-point contraction off (integer decisions depend on
// one rounding per operation).
#include <type_traits>

#include "pod_internal.h"
#include "pod_tile.h"
#include "pod_trade.h"

namespace pod {

namespace {

using namespace tile;
using O = Op<false>;

constexpr int NM = 4, NE = 4;       // wavefronts of the network / of the envs
constexpr int NT = 64 * (NM + NE);
constexpr int HP = tile_pitch<false>(16);
constexpr int MUP = 36;             // row pitch of a plane of partial means
constexpr int LB = 8 * 192;         // 16-byte pieces of a k-block of a hidden layer

// What differs between 16 and 32 envs: the matrix instruction, and with it how weights, inputs and sums lie in the lanes.
//  32: v_mfma_f32_32x32x16, lane l feeds feature l % 32 and row l % 32, inputs 8 (l / 32) .. + 7 of 16
//  16: v_mfma_f32_16x16x32, lane l feeds feature l % 16 and row l % 16, inputs 8 (l / 16) .. + 7 of 32
// A unit is such an operand of the packed weights, whose blocks are made for the first: for 16 envs, half the features of
// two blocks.  A lane holds sums of its row for groups of four features.
template <int E>
struct Geometry {
  static constexpr bool SM = E == 16;
  typedef std::conditional_t<SM, f32x4, f32x16> Acc;
  static constexpr int NACC = SM ? 4 : 2;             // accumulators of a wavefront's 64 features: units per block of inputs
  static constexpr int KIN = SM ? 32 : 16;            // inputs per block
  static constexpr int KBYTES = KIN * O::ESZ;         // ... in an activation row
  static constexpr int BLOCK = SM ? 2 * LB : LB;      // 16-byte pieces between the blocks of a hidden layer
  static constexpr int NK2 = 256 / KIN;
  static constexpr int PK = SM ? 2 : 4, PU = PK * NACC;  // blocks, and units of weights, in flight per wavefront
  static constexpr int NL = SM ? 7 : 1;               // units of layer 2 per wavefront that stay in LDS
  static constexpr int NG = SM ? 4 : 8;               // groups of four features per lane
  static constexpr int N3 = SM ? 2 : 4, NC3 = SM ? 2 : 1;  // output layer: blocks of a wavefront's inputs, tiles of outputs
  static constexpr int ND = E / 8, ROWS = E / NE;     // stocks per thread and market rows per wavefront of the envs
  static constexpr int PLANE = E * MUP;
  using Tr = Trade<E, ND, true, 64 * NE>;

  static __device__ inline int row(int lane) { return lane & (E - 1); }
  static __device__ inline int part(int lane) { return lane / E; }
  static __device__ inline const u32x4 *base(const u32x4 *W, int w, int lane) {  // of unit 0 of features 64 w ..
    return SM ? W + ((size_t)(lane >> 5) * 8 + 2 * w) * 192 + ((lane >> 4) & 1) * 32 + (lane & 15) : W + (size_t)(2 * w) * 192 + lane;
  }
  static __device__ inline const u32x4 *unit(const u32x4 *W, int u) {
    return W + (size_t)(u / NACC) * BLOCK + (SM ? ((u >> 1) & 1) * 192 + (u & 1) * 16 : (u & 1) * 192);
  }
  static __device__ inline void fetch_unit(Blk3 &b, const u32x4 *W, int u) { fetch_w(b, unit(W, u)); }
  static __device__ inline void mma(const Blk3 &w, const Blk3 &x, Acc &c) {
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      const bf16x8 a = __builtin_bit_cast(bf16x8, w.p[kSplitA[i]]), b = __builtin_bit_cast(bf16x8, x.p[kSplitB[i]]);
      if constexpr (SM) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
      else c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
  }
  static __device__ inline void clear(Acc &c) {
#pragma unroll
    for (int i = 0; i < (SM ? 4 : 16); ++i) c[i] = 0.0f;
  }
  // group m of a wavefront's features: its first feature (of lane part q), and its sums
  static __device__ inline int feature(int m, int q) { return (SM ? 16 : 8) * m + 4 * q; }
  static __device__ inline float get(const Acc (&c)[NACC], int m, int i) { return SM ? c[m][i] : c[m >> 2][4 * (m & 3) + i]; }
  static __device__ inline void put(Acc (&c)[NACC], int m, int i, float v) {
    if (SM) c[m][i] = v;
    else c[m >> 2][4 * (m & 3) + i] = v;
  }
};

// whole blocks of 32 inputs for the short instruction
template <int E>
__host__ __device__ inline int input_pitch(int S) { return tile_pitch<false>(E == 16 ? (S + 31) / 32 * 2 : (S + 15) / 16); }

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

// tanh of sixteen values, one operation at a time over all of them (see tanh_in_place), with between(0 .. 11) behind each.
template <class Between>
__device__ inline void tanh_accurate_16(float (&z)[16], Between between) {
  float e[16], x2[16], ps[16];
  int stage = 0;
  auto all = [&](auto op) {
#pragma unroll
    for (int i = 0; i < 16; ++i) op(i, z[i]);
    between(stage++);
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
  all([&](int i, float x) { z[i] = fabsf(x) < 0.25f ? ps[i] : e[i]; });
}

// acc += blocks [0, n) of a range of inputs; the ring holds the first units.  N > 0: n at compile time, in straight-line code.
template <class G, int N>
__device__ inline void products(typename G::Acc (&acc)[G::NACC], Blk3 (&ring)[G::PU], const unsigned char *x, const u32x4 *W, int n) {
  if constexpr (N > 0) {
    Blk3 xn;
    fetch_x(xn, x);
#pragma unroll
    for (int K = 0; K < N; ++K) {
      const Blk3 xv = xn;
#pragma unroll
      for (int j = 0; j < G::NACC; ++j) {
        const int u = G::NACC * K + j;
        if (j == 0 && K + 1 < N) {
          fetch_x(xn, x + (K + 1) * G::KBYTES);
          __builtin_amdgcn_sched_barrier(0);
        }
        G::mma(ring[u % G::PU], xv, acc[j]);
        if (u + G::PU < G::NACC * N) G::fetch_unit(ring[u % G::PU], W, u + G::PU);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  } else {
    auto block = [&](int K, int k) {  // (k: K modulo PK, at compile time)
      Blk3 xv;
      fetch_x(xv, x + K * G::KBYTES);
#pragma unroll
      for (int j = 0; j < G::NACC; ++j) {
        G::mma(ring[G::NACC * k + j], xv, acc[j]);
        G::fetch_unit(ring[G::NACC * k + j], W, G::NACC * min(K + G::PK, n - 1) + j);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    int K = 0;
    for (; K + G::PK <= n; K += G::PK) {
#pragma unroll
      for (int k = 0; k < G::PK; ++k) block(K + k, k);
    }
#pragma unroll
    for (int k = 0; k < G::PK - 1; ++k)
      if (K + k < n) block(K + k, k);
  }
}

// Layer 2: the first NL units from LDS (`own`, this lane's), the others through the ring, which holds the first of them.
template <class G>
__device__ inline void products2(typename G::Acc (&acc)[G::NACC], Blk3 (&ring)[G::PU], const unsigned char *x, const u32x4 *own, const u32x4 *W) {
  constexpr int NL = G::NL;
  Blk3 xn, wn;
  fetch_x(xn, x);
  fetch_w(wn, own);
#pragma unroll
  for (int K = 0; K < G::NK2; ++K) {
    const Blk3 xv = xn;
#pragma unroll
    for (int j = 0; j < G::NACC; ++j) {
      const int u = G::NACC * K + j, r = u - NL;
      const Blk3 wv = r < 0 ? wn : ring[r < 0 ? 0 : r % G::PU];
      if (j == 0 && K + 1 < G::NK2) fetch_x(xn, x + (K + 1) * G::KBYTES);
      if (u + 1 < NL) fetch_w(wn, own + (u + 1) * 192);
      __builtin_amdgcn_sched_barrier(0);
      G::mma(wv, xv, acc[j]);
      if (r >= 0 && u + G::PU < G::NACC * G::NK2) G::fetch_unit(ring[r % G::PU], W, u + G::PU);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// NK1, NH: blocks of layer 1, and how many of them hold market columns only (0: at run time)
template <int E, int NK1, int NH>
__global__ __launch_bounds__(NT, 2) void rollout_f32_kernel(F32Args a) {
  using G = Geometry<E>;
  using Tr = typename G::Tr;
  constexpr int PLANE = G::PLANE, TPE = Tr::TPE, ND = G::ND, ROWS = G::ROWS, PU = G::PU, NL = G::NL;
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
    const int nk1 = NK1 > 0 ? NK1 : (S + G::KIN - 1) / G::KIN, nh = NH > 0 ? NH : (DK + D) / G::KIN;
    const int row = G::row(lane), part = G::part(lane);
    const unsigned char *xrow = ldsX + row * a.xpitch + O::HALF * part, *hrow = ldsH + row * HP + O::HALF * part;
    Blk3 ring[PU];
    typename G::Acc acc[G::NACC];
    auto prime_range = [&](const u32x4 *W, int n) {
#pragma unroll
      for (int u = 0; u < PU; ++u)
        if (u / G::NACC < n) G::fetch_unit(ring[u], W, u);
    };
    auto clear = [&]() {
#pragma unroll
      for (int j = 0; j < G::NACC; ++j) G::clear(acc[j]);
    };
    // tanh of the sums, and between its operations, part by part, the ring is filled: all at once the
    // requests take longer to issue than they take to be answered (2 us for 24 KB a wavefront, the vector units idle)
    auto activate = [&](const float *bias, auto unit_of_next) {
      constexpr int PER = 3 * PU * 4 / (12 * G::NG);
#pragma unroll
      for (int m0 = 0; m0 < G::NG; m0 += 4) {
        float z[16];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          const f32x4 b = *reinterpret_cast<const f32x4 *>(bias + 64 * w + G::feature(m0 + m, part));
#pragma unroll
          for (int i = 0; i < 4; ++i) z[4 * m + i] = G::get(acc, m0 + m, i) + b[i];
        }
        tanh_accurate_16(z, [&](int stage) {
#pragma unroll
          for (int k = 0; k < PER; ++k) {
            const int p = (stage + 3 * m0) * PER + k;
            ring[p / 3].p[p % 3] = unit_of_next(p / 3)[64 * (p % 3)];
          }
        });
#pragma unroll
        for (int m = 0; m < 16; ++m) G::put(acc, m0 + (m >> 2), m & 3, z[m]);
      }
    };
    int lane_s = lane;
    const u32x4 *W1, *W2;
    auto addresses = [&]() {  // (opaque per step, or the addresses of all weight blocks are kept across the steps)
      asm volatile("" : "+v"(lane_s));
      W1 = G::base(net.W[0], w, lane_s);
      W2 = G::base(net.W[1], w, lane_s);
    };
    auto head = [&]() {
      clear();
      products<G, NH>(acc, ring, xrow, W1, nh);
      prime_range(W1 + (size_t)nh * G::BLOCK, nk1 - nh);
    };
    addresses();
    // kept: the first units of layer 2 (LDS) and the output layer's weights (registers).  A lane of that layer's operand
    // takes the two halves of its piece from the places the order of its inputs has them in (see below).
    u32x4 *own = ldsW + (size_t)w * (NL * 192) + lane;
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      Blk3 b;
      G::fetch_unit(b, W2, u);
#pragma unroll
      for (int i = 0; i < 3; ++i) own[u * 192 + 64 * i] = b.p[i];
    }
    const unsigned char *W3 = reinterpret_cast<const unsigned char *>(net.W[2] + (size_t)w * (4 * 192) + (E == 16 ? (part >> 1) * 32 : 0) + row) + 8 * (part & 1);
    constexpr int W3K = E == 16 ? 2 * 192 : 192, W3H = E == 16 ? 192 : 32;  // pieces from block to block, and to the second half
    Blk3 w3[G::N3][G::NC3];
#pragma unroll
    for (int K = 0; K < G::N3; ++K)
#pragma unroll
      for (int c = 0; c < G::NC3; ++c)
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          const u32x2 lo = *reinterpret_cast<const u32x2 *>(W3 + (K * W3K + c * 16 + i * 64) * 16);
          const u32x2 hi = *reinterpret_cast<const u32x2 *>(W3 + (K * W3K + W3H + c * 16 + i * 64) * 16);
          w3[K][c].p[i] = u32x4{lo[0], lo[1], hi[0], hi[1]};
        }
    prime_range(W1, nh);
    __syncthreads();  // observation 0 complete
    head();
    for (int t = 0; t < a.T; ++t) {
      __syncthreads();  // observation t complete
      {
        // (sums of their own, like the output layer's below)
        typename G::Acc head_sums[G::NACC];
#pragma unroll
        for (int j = 0; j < G::NACC; ++j) head_sums[j] = acc[j];
        clear();
        products<G, NK1 - NH>(acc, ring, xrow + nh * G::KBYTES, W1 + (size_t)nh * G::BLOCK, nk1 - nh);
#pragma unroll
        for (int j = 0; j < G::NACC; ++j) acc[j] += head_sums[j];
      }
      addresses();
      activate(ldsBias, [&](int u) { return G::unit(W2, NL + u); });
#pragma unroll
      for (int m = 0; m < G::NG; ++m)
        O::store4<true>(ldsH + row * HP + O::off(64 * w + G::feature(m, part)), G::get(acc, m, 0), G::get(acc, m, 1), G::get(acc, m, 2),
                        G::get(acc, m, 3));
      __syncthreads();  // first hidden layer complete, input tile free
      clear();
      products2<G>(acc, ring, hrow, own, W2);
      // Output layer, from registers: the eight values a lane holds of two groups of features are an operand of the
      // transposed product in another order of its inputs.  Each wavefront adds up its own features for all outputs.
      const int last_head = max(nh - 1, 0);
      activate(ldsBias + 256, [&](int u) { return G::unit(W1, NH > 0 ? u : G::NACC * min(u / G::NACC, last_head) + u % G::NACC); });
      // (each block's sums start at zero and are added to the others afterwards: one chain over all leaves a larger error, 16
      // envs, 2-norm of the means 3.16e-7 for 3.06e-7)
      typename G::Acc o[G::NC3];
#pragma unroll
      for (int K = 0; K < G::N3; ++K) {
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = G::get(acc, 2 * K + (i >> 2), i & 3);
        bf16x8 xs[3];
        split3<true>(v, xs);
        Blk3 xv;
#pragma unroll
        for (int i = 0; i < 3; ++i) xv.p[i] = __builtin_bit_cast(u32x4, xs[i]);
#pragma unroll
        for (int c = 0; c < G::NC3; ++c) {
          typename G::Acc p;
          G::clear(p);
          G::mma(w3[K][c], xv, p);
          o[c] = K == 0 ? p : o[c] + p;
        }
      }
      float *plane = planes + w * PLANE + row * MUP;
#pragma unroll
      for (int m = 0; m < (E == 16 ? 2 : 4); ++m) {
        f32x4 v;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = o[E == 16 ? m : 0][(E == 16 ? 0 : 4 * m) + i];
        *reinterpret_cast<f32x4 *>(plane + G::feature(m, part)) = v;
      }
      __syncthreads();  // means and the market columns of observation t + 1 complete
      if (t + 1 < a.T) head();
    }
    return;
  }

  // ------------------------------------------------------------------ the envs
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
    __builtin_amdgcn_s_setprio(3);  // (from here to the next observation the network can wait, elsewhere the envs)
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
    __builtin_amdgcn_s_setprio(0);
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

template <int E>
size_t lds_bytes(int S) {
  using G = Geometry<E>;
  return (size_t)E * (input_pitch<E>(S) + HP) + ((size_t)NM * G::PLANE + (2 * 256 + 32)) * 4 + (size_t)E * 32 * 8 + (size_t)NM * G::NL * 3072;
}

template <int E, int NK1, int NH>
hipError_t launch_inst(hipStream_t st, const F32Args &a, size_t lds) {
  constexpr auto kern = rollout_f32_kernel<E, NK1, NH>;
  const hipError_t e = allow_full_lds<kern>();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)(a.d.N / E)), dim3(NT), lds, st, a);
  return hipGetLastError();
}

template <int E, int NK1, int NH>
hipError_t launch_geometry(hipStream_t st, F32Args a) {
  const EnvDims &d = a.d;
  a.xpitch = input_pitch<E>(d.S);
  const size_t lds = lds_bytes<E>(d.S);
  if (d.N % E || a.envs_per_agent % E || trade_lds(E, true, d.D) > (size_t)E * HP || lds > (size_t)kMaxLdsBytes) return hipErrorInvalidValue;
  constexpr int KIN = Geometry<E>::KIN;
  // Layer 1 in straight-line code, each block's inputs read a block ahead, for the blocks of 30 stocks x 8 indicators (289 to
  // 320 or 304 inputs, 256 to 287 or 271 of them market columns).  us a step with numbers of blocks at run time and this:
  // 16 envs, where layer 1 is a third of the chain, 1024 envs 9.7 -> 8.0, 4096 12.2 -> 9.9; 32 envs 65536 of 64 agents 0.4
  // and 1.2 % on two chips, 8192 and 16384 level.
  if ((d.S + KIN - 1) / KIN == NK1 && (d.D * d.K + d.D) / KIN == NH) return launch_inst<E, NK1, NH>(st, a, lds);
  return launch_inst<E, 0, 0>(st, a, lds);
}

// 16 envs up to a workgroup for each of the 256 compute units; beyond, the weights streamed once for 32 envs are worth
// more (301 inputs, per step: 4096 envs 10.9 us against 14.1, 1024 8.2 against 13.0; 8192 in two rounds 21 against 17.2).
bool sixteen(int N) { return N <= 256 * 16; }

}  // namespace

size_t fused_f32_lds_bytes(const pr_config &c) {
  const int S = 1 + 2 * c.n_stocks + c.n_stocks * c.n_ind;
  return sixteen(c.n_envs) ? lds_bytes<16>(S) : lds_bytes<32>(S);
}

hipError_t launch_rollout_fused_f32(hipStream_t st, const EnvDims &d, const EnvState &s, const float *price, const float *ind,
                                    const PackedNet &actor, int32_t envs_per_agent, int32_t T, const float *noise,
                                    const pr_buffers &out) {
  F32Args a;
  a.d = d, a.st = s, a.price = price, a.ind = ind, a.actor = actor, a.envs_per_agent = envs_per_agent, a.T = T;
  a.noise = noise, a.obs = out.obs, a.act_raw = out.act_raw, a.reward = out.reward, a.done = out.done, a.logp = out.logp;
  a.mu_out = out.mu, a.shares = out.shares;
  if (actor.bf16 || actor.nkb[0] % 2 || actor.nkb[1] != 16 || actor.nct[0] != 8 || actor.nct[2] != 1) return hipErrorInvalidValue;
  return sixteen(d.N) ? launch_geometry<16, 10, 8>(st, a) : launch_geometry<32, 19, 16>(st, a);
}

}  // namespace pod
