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
// Hidden layers and the market part of layer 1 are products of two fp16 parts per operand (pod_half2.h): half the matrix
// work and two thirds of the weights' bytes of three bf16 parts.  A row's market columns have a scale of their own, found while
// they are written beside layer 2.  The portfolio's columns come at the end of the trades and are a block or two: there three
// bf16 parts, which need no scale, cost less than a search for one.
//
// Bound with 16 envs by the chain of a step -- tail of layer 1, activation, layer 2, activation, output layer, trades of 3 us --
// beside a weight stream of 510 KB (96 KB of layer 2 stay in LDS, the output layer's 32 KB in registers), 4.2 us at 64 B a
// clock; with 32 envs by vector work (1700 instructions a wavefront and step, 49 % of the cycles) and the same chain, the
// matrix pipe busy 27 % at 1.85 GHz.
// 301 inputs, per step, against three bf16 parts in all products: 1024 envs 8.1 -> 6.6 us, 4096 9.9 -> 7.9, 8192 17.0 ->
// 14.2, 16384 33.6 -> 27.6, 65536 of 64 agents 139 -> 110; 12 stocks x 4 indicators, 4096 envs 8.6 -> 6.0, 8192 11.7 -> 10.1.
// 2-norm of the means' error against 64 bits: 4096 envs 3.02e-7 -> 2.72e-7, 8192 3.12 -> 2.80, 1024 envs of 8 stocks x 4
// indicators 2.19 -> 2.10 (2.26 with layer 2 in one chain over all inputs, not in two halves added up).
//
// Compiled with floating-point contraction off (integer decisions depend on
// one rounding per operation).
#include <type_traits>

#include "pod_half2.h"
#include "pod_internal.h"
#include "pod_tile.h"
#include "pod_trade.h"

namespace pod {

namespace {

using namespace tile;
using O = Op<false>;

constexpr int NM = 4, NE = 4;       // wavefronts of the network / of the envs
constexpr int NT = 64 * (NM + NE);
constexpr int MUP = 36;             // row pitch of a plane of partial means

// An operand of the hidden layers, eight consecutive inputs of a row or a feature: their two fp16 parts.
struct Blk2 {
  u32x4 p[2];
};
// ... in an activation row: 16 bytes of first parts, 16 of second ones; where column c starts
__host__ __device__ inline int half_off(int c) { return (c >> 3) * 32 + (c & 7) * 2; }
__host__ __device__ constexpr int half_pitch(int nkb) { return nkb * 64 + 16; }
constexpr int HP = half_pitch(16);

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
  static constexpr int KBYTES = KIN * 4;              // ... in an activation row of fp16 parts
  static constexpr int BLOCK = (SM ? 2 : 1) * 8 * 128;  // 16-byte pieces between the blocks of a hidden layer
  static constexpr int PBLOCK = (SM ? 2 : 1) * 8 * 192, PBYTES = KIN * O::ESZ;  // ... and of its part in three bf16 numbers
  static constexpr int NK2 = 256 / KIN;
  static constexpr int PK = SM ? 3 : 6, PU = PK * NACC;  // blocks, and units of weights, in flight per wavefront
  static constexpr int NP = SM ? 2 : 3;               // blocks of portfolio columns at most
  static constexpr int NL = SM ? 12 : 5;              // units of layer 2 per wavefront that stay in LDS
  static constexpr int NG = SM ? 4 : 8;               // groups of four features per lane
  static constexpr int N3 = SM ? 2 : 4, NC3 = SM ? 2 : 1;  // output layer: blocks of a wavefront's inputs, tiles of outputs
  static constexpr int ND = E / 8, ROWS = E / NE;     // stocks per thread and market rows per wavefront of the envs
  static constexpr int PLANE = E * MUP;
  using Tr = Trade<E, ND, true, 64 * NE>;

  static __device__ inline int row(int lane) { return lane & (E - 1); }
  static __device__ inline int part(int lane) { return lane / E; }
  // of unit 0 of features 64 w .., in blocks of PIECES 16-byte pieces
  template <int PIECES>
  static __device__ inline const u32x4 *base(const u32x4 *W, int w, int lane) {
    return SM ? W + ((size_t)(lane >> 5) * 8 + 2 * w) * PIECES + ((lane >> 4) & 1) * 32 + (lane & 15) : W + (size_t)(2 * w) * PIECES + lane;
  }
  static __device__ inline const u32x4 *unit(const u32x4 *W, int u) {
    return W + (size_t)(u / NACC) * BLOCK + (SM ? ((u >> 1) & 1) * 128 + (u & 1) * 16 : (u & 1) * 128);
  }
  static __device__ inline const u32x4 *unit3(const u32x4 *W, int u) {
    return W + (size_t)(u / NACC) * PBLOCK + (SM ? ((u >> 1) & 1) * 192 + (u & 1) * 16 : (u & 1) * 192);
  }
  static __device__ inline void mma(const Blk2 &w, const Blk2 &x, Acc &c) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {  // the smallest first
      const f16x8 a = __builtin_bit_cast(f16x8, w.p[i == 0]), b = __builtin_bit_cast(f16x8, x.p[i == 1]);
      if constexpr (SM) c = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
      else c = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
    }
  }
  static __device__ inline void mma3(const u32x4 *w, const Blk3 &x, Acc &c) {
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      const bf16x8 a = __builtin_bit_cast(bf16x8, w[kSplitA[i]]), b = __builtin_bit_cast(bf16x8, x.p[kSplitB[i]]);
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

__device__ inline void fetch_half(Blk2 &b, const u32x4 *p) { b.p[0] = p[0], b.p[1] = p[64]; }
__device__ inline void fetch_half(Blk2 &b, const unsigned char *p) {
  b.p[0] = *reinterpret_cast<const u32x4 *>(p), b.p[1] = *reinterpret_cast<const u32x4 *>(p + 16);
}
__device__ inline void put_half4(unsigned char *p, const float (&v)[4]) {  // (scaled tanh outputs)
  uint32_t h0, h1, l0, l1;
  split2_pair<true>(v[0], v[1], h0, l0);
  split2_pair<true>(v[2], v[3], h1, l1);
  *reinterpret_cast<u32x2 *>(p) = u32x2{h0, h1};
  *reinterpret_cast<u32x2 *>(p + 16) = u32x2{l0, l1};
}

// the largest of the wavefront's numbers, none of which is negative
__device__ inline float wave_max(float x) {
  int v = __builtin_bit_cast(int, x);
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true));  // one, two, four, eight lanes of a row of 16 over
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true));
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true));
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true));
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, true));  // the last lane of a row to the next row, of two to the next two
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, true));
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(v, 63));
}

struct F32Args {
  EnvDims d;
  EnvState st;
  const float *price, *ind;
  PackedNet actor;  // layer 1 in the input order [indicators | prices | zeros | holdings | cash | zeros], either part in whole
                    // blocks of 32 inputs; in fp16 parts its market part and the other layers
  int32_t envs_per_agent, T;
  int32_t market, portfolio;  // k-blocks of either part
  int32_t hidden_bytes;       // of the hidden tile's place, which the trades take as well
  const float *noise;  // [T, N, D]
  float *obs;          // [T+1, N, S]
  float *act_raw;      // [T, N, D]
  float *reward;       // [T, N]
  uint8_t *done;       // [T, N]
  float *logp;         // opt [T, N]
  float *mu_out;       // opt [T, N, D]
  int32_t *shares;     // opt [T, N, D]
};

// tanh of sixteen values, times kHiddenScale, one operation at a time over all of them (see tanh_in_place), with between(0 .. 11)
// behind each.
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
  all([&](int i, float x) { e[i] = copysignf(fmaf(e[i], -2.0f * kHiddenScale, kHiddenScale), x), ps[i] = ps[i] * kHiddenScale; });
  all([&](int i, float x) { z[i] = fabsf(x) < 0.25f ? ps[i] : e[i]; });
}

// acc += blocks [0, n) of a range of inputs; the ring holds the first units.  N > 0: n at compile time, in straight-line code.
template <class G, int N>
__device__ inline void products(typename G::Acc (&acc)[G::NACC], Blk2 (&ring)[G::PU], const unsigned char *x, const u32x4 *W, int n) {
  if constexpr (N > 0) {
    Blk2 xn;
    fetch_half(xn, x);
#pragma unroll
    for (int K = 0; K < N; ++K) {
      const Blk2 xv = xn;
#pragma unroll
      for (int j = 0; j < G::NACC; ++j) {
        const int u = G::NACC * K + j;
        if (j == 0 && K + 1 < N) {
          fetch_half(xn, x + (K + 1) * G::KBYTES);
          __builtin_amdgcn_sched_barrier(0);
        }
        G::mma(ring[u % G::PU], xv, acc[j]);
        if (u + G::PU < G::NACC * N) fetch_half(ring[u % G::PU], G::unit(W, u + G::PU));
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  } else {
    auto block = [&](int K, int k) {  // (k: K modulo PK, at compile time)
      Blk2 xv;
      fetch_half(xv, x + K * G::KBYTES);
#pragma unroll
      for (int j = 0; j < G::NACC; ++j) {
        G::mma(ring[G::NACC * k + j], xv, acc[j]);
        fetch_half(ring[G::NACC * k + j], G::unit(W, G::NACC * min(K + G::PK, n - 1) + j));
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

// Layer 2, in two chains over half of the inputs each: the first NL units from LDS (`own`, this lane's), the others through the ring, which holds the first of them.
template <class G>
__device__ inline void products2(typename G::Acc (&acc)[G::NACC], Blk2 (&ring)[G::PU], const unsigned char *x, const u32x4 *own, const u32x4 *W) {
  constexpr int NL = G::NL;
  typename G::Acc first[G::NACC];
  Blk2 xn, wn;
  fetch_half(xn, x);
  fetch_half(wn, own);
#pragma unroll
  for (int K = 0; K < G::NK2; ++K) {
    const Blk2 xv = xn;
#pragma unroll
    for (int j = 0; j < G::NACC; ++j) {
      if (K == G::NK2 / 2) {
        first[j] = acc[j];
        G::clear(acc[j]);
      }
      const int u = G::NACC * K + j, r = u - NL;
      const Blk2 wv = r < 0 ? wn : ring[r < 0 ? 0 : r % G::PU];
      if (j == 0 && K + 1 < G::NK2) fetch_half(xn, x + (K + 1) * G::KBYTES);
      if (u + 1 < NL) fetch_half(wn, own + (u + 1) * 128);
      __builtin_amdgcn_sched_barrier(0);
      G::mma(wv, xv, acc[j]);
      if (r >= 0 && u + G::PU < G::NACC * G::NK2) fetch_half(ring[r % G::PU], G::unit(W, u + G::PU));
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int j = 0; j < G::NACC; ++j) acc[j] += first[j];
}

// NH, NP: blocks of market and of portfolio columns (0: at run time)
template <int E, int NH, int NP>
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
  const int xpitch = half_pitch(a.market), ppitch = tile_pitch<false>(a.portfolio);
  unsigned char *ldsX = lds, *ldsP = ldsX + E * xpitch;     // input tile: market columns, scaled and in fp16 parts, and portfolio
  unsigned char *ldsH = ldsP + E * ppitch;                  // hidden tile, and in it the trades' scratch
  float *planes = reinterpret_cast<float *>(ldsH + a.hidden_bytes);  // [NM][E][MUP] partial means
  float *ldsBias = planes + NM * PLANE;                     // b1 | b2 | b3
  float *ldsU = ldsBias + 2 * 256 + 32;                     // factors of the three layers' features
  float *rowU = ldsU + 2 * 256 + 32;                        // [E] and of the market part of layer 1's rows
  double *ldsTerms = reinterpret_cast<double *>(rowU + E);  // holdings' values, read while the hidden tile is in use
  u32x4 *ldsW = reinterpret_cast<u32x4 *>(ldsTerms + E * 32);
  const int agent = (n0 % d.N) / a.envs_per_agent;
  const Net net = net_of(a.actor, agent);
  auto half_w = [&](int l, int nkb, int nct) {
    return reinterpret_cast<const u32x4 *>(static_cast<const unsigned char *>(a.actor.half_w[l]) + agent * halves_bytes(nkb, nct));
  };

  for (int i = tid; i < E * (xpitch + ppitch) / 4; i += NT) reinterpret_cast<uint32_t *>(ldsX)[i] = 0u;  // (padded k columns stay so)
  if (tid < 256) ldsU[tid] = a.actor.half_u[0][(size_t)agent * 256 + tid];
  else ldsU[tid] = a.actor.half_u[1][(size_t)agent * 256 + tid - 256];
  if (tid < 32) ldsU[512 + tid] = a.actor.half_u[2][(size_t)agent * 32 + tid];
  stage_net<NT>(net, ldsBias, nullptr, tid);
  __syncthreads();

  if (w < NM) {
    // ---------------------------------------------------------------- the network, features 64 w ..
    const int nh = NH > 0 ? NH : (DK + D + G::KIN - 1) / G::KIN, np = NP > 0 ? NP : (D + G::KIN) / G::KIN;
    const int row = G::row(lane), part = G::part(lane);
    const unsigned char *xrow = ldsX + row * xpitch + 32 * part, *prow = ldsP + row * ppitch + O::HALF * part, *hrow = ldsH + row * HP + 32 * part;
    Blk2 ring[PU];  // (for the portfolio part of layer 1 all of its blocks)
    typename G::Acc acc[G::NACC];
    auto prime_range = [&](const u32x4 *W, int n) {
#pragma unroll
      for (int u = 0; u < PU; ++u)
        if (u / G::NACC < n) fetch_half(ring[u], G::unit(W, u));
    };
    auto clear = [&]() {
#pragma unroll
      for (int j = 0; j < G::NACC; ++j) G::clear(acc[j]);
    };
    // tanh of the sums, and between its operations, part by part, the ring is filled: all at once the
    // requests take longer to issue than they take to be answered (2 us for 24 KB a wavefront, the vector units idle)
    auto activate = [&](int layer, auto unit_of_next) {
      constexpr int PER = 2 * PU * 4 / (12 * G::NG);
      static_assert(PER * 12 * G::NG == 2 * PU * 4, "");
#pragma unroll
      for (int m0 = 0; m0 < G::NG; m0 += 4) {
        float z[16];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          const int f = 256 * layer + 64 * w + G::feature(m0 + m, part);
          const f32x4 b = *reinterpret_cast<const f32x4 *>(ldsBias + f), u = *reinterpret_cast<const f32x4 *>(ldsU + f);
#pragma unroll
          for (int i = 0; i < 4; ++i)  // (layer 1's sums have their factors already)
            z[4 * m + i] = layer == 0 ? G::get(acc, m0 + m, i) + b[i] : fmaf(G::get(acc, m0 + m, i), u[i], b[i]);
        }
        tanh_accurate_16(z, [&](int stage) {
#pragma unroll
          for (int k = 0; k < PER; ++k) {
            const int p = (stage + 3 * m0) * PER + k;
            ring[p / 2].p[p % 2] = unit_of_next(p / 2)[64 * (p % 2)];
          }
        });
#pragma unroll
        for (int m = 0; m < 16; ++m) G::put(acc, m0 + (m >> 2), m & 3, z[m]);
      }
    };
    int lane_s = lane;
    const u32x4 *W1, *W1p, *W2;
    auto addresses = [&]() {  // (opaque per step, or the addresses of all weight blocks are kept across the steps)
      asm volatile("" : "+v"(lane_s));
      W1 = G::template base<128>(half_w(0, a.market, 8), w, lane_s);
      W1p = G::template base<192>(net.W[0] + (size_t)a.market * (8 * 192), w, lane_s);
      W2 = G::template base<128>(half_w(1, 16, 8), w, lane_s);
    };
    // Market part of layer 1: its rows and weights are scaled, what it adds up is not any more.  Behind it the ring takes the
    // weights of the portfolio part, three pieces a unit.
    auto piece = [&](int i) -> u32x4 & { return ring[i / 2].p[i % 2]; };
    static_assert(3 * G::NP * G::NACC <= 2 * PU, "");
    auto head = [&]() {
      clear();
      products<G, NH>(acc, ring, xrow, W1, nh);
#pragma unroll
      for (int u = 0; u < G::NP * G::NACC; ++u)
        if (u / G::NACC < np)
#pragma unroll
          for (int i = 0; i < 3; ++i) piece(3 * u + i) = G::unit3(W1p, u)[64 * i];
      const float ru = rowU[row];
#pragma unroll
      for (int m = 0; m < G::NG; ++m) {
        const f32x4 u = *reinterpret_cast<const f32x4 *>(ldsU + 64 * w + G::feature(m, part));
#pragma unroll
        for (int i = 0; i < 4; ++i) G::put(acc, m, i, G::get(acc, m, i) * ru * u[i]);
      }
    };
    addresses();
    // kept: the first units of layer 2 (LDS) and the output layer's weights (registers).  A lane of that layer's operand
    // takes the two halves of its piece from the places the order of its inputs has them in (see below).
    u32x4 *own = ldsW + (size_t)w * (NL * 128) + lane;
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      Blk2 b;
      fetch_half(b, G::unit(W2, u));
#pragma unroll
      for (int i = 0; i < 2; ++i) own[u * 128 + 64 * i] = b.p[i];
    }
    const unsigned char *W3 = reinterpret_cast<const unsigned char *>(half_w(2, 16, 1) + (size_t)w * (4 * 128) + (E == 16 ? (part >> 1) * 32 : 0) + row) + 8 * (part & 1);
    constexpr int W3K = E == 16 ? 2 * 128 : 128, W3H = E == 16 ? 128 : 32;  // pieces from block to block, and to the second half
    Blk2 w3[G::N3][G::NC3];
#pragma unroll
    for (int K = 0; K < G::N3; ++K)
#pragma unroll
      for (int c = 0; c < G::NC3; ++c)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
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
#pragma unroll
        for (int K = 0; K < G::NP; ++K)
          if (K < np) {
            Blk3 xv;
            fetch_x(xv, prow + K * G::PBYTES);
#pragma unroll
            for (int j = 0; j < G::NACC; ++j) {
              const int u = 3 * (G::NACC * K + j);
              const u32x4 wv[3] = {piece(u), piece(u + 1), piece(u + 2)};
              G::mma3(wv, xv, acc[j]);
            }
          }
#pragma unroll
        for (int j = 0; j < G::NACC; ++j) acc[j] += head_sums[j];
      }
      addresses();
      activate(0, [&](int u) { return G::unit(W2, NL + u); });
#pragma unroll
      for (int m = 0; m < G::NG; ++m)
      {
        const float v[4] = {G::get(acc, m, 0), G::get(acc, m, 1), G::get(acc, m, 2), G::get(acc, m, 3)};
        put_half4(ldsH + row * HP + half_off(64 * w + G::feature(m, part)), v);
      }
      __syncthreads();  // first hidden layer complete, input tile free
      clear();
      products2<G>(acc, ring, hrow, own, W2);
      // Output layer, from registers: the eight values a lane holds of two groups of features are an operand of the
      // transposed product in another order of its inputs.  Each wavefront adds up its own features for all outputs.
      const int last_head = nh - 1;
      activate(1, [&](int u) { return G::unit(W1, NH > 0 ? u : G::NACC * min(u / G::NACC, last_head) + u % G::NACC); });
      // (each block's sums start at zero and are added to the others afterwards: one chain over all leaves a larger error, 16
      // envs, 2-norm of the means 3.16e-7 for 3.06e-7)
      typename G::Acc o[G::NC3];
#pragma unroll
      for (int K = 0; K < G::N3; ++K) {
        Blk2 xv;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          uint32_t hi, lo;
          split2_pair<true>(G::get(acc, 2 * K + (i >> 1), 2 * (i & 1)), G::get(acc, 2 * K + (i >> 1), 2 * (i & 1) + 1), hi, lo);
          xv.p[0][i] = hi, xv.p[1][i] = lo;
        }
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
  const float *lb3 = ldsBias + 2 * 256, *lu3 = ldsU + 2 * 256;
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
  unsigned char *penv = ldsP + e * ppitch;
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
      unsigned char *x = ldsX + er * xpitch;
      const float pv = r_p[j] * d.s_price;
      __builtin_nontemporal_store(pv, &orow[1 + lp]);
      f32x4 v = r_i[j];
      v[0] *= d.s_ind, v[1] *= d.s_ind, v[2] *= d.s_ind, v[3] *= d.s_ind;
      // observation rows are 4-byte aligned only; a 16-byte store needs no more than that
      __builtin_nontemporal_store(v, reinterpret_cast<f32x4 *>(orow + 1 + 2 * D) + li);
      // The tile has the row over the power of two of its largest finite number, which goes to 2^14 .. 2^15.
      auto finite = [](float f) { return fabsf(f) < __builtin_inff() ? fabsf(f) : 0.0f; };
      const float m = wave_max(fmaxf(fmaxf(fmaxf(finite(v[0]), finite(v[1])), fmaxf(finite(v[2]), finite(v[3]))), finite(pv)));
      const uint32_t me = min(max(__builtin_bit_cast(uint32_t, m > 0.0f ? m : 1.0f) >> 23, 15u), 254u);
      const float scale = __builtin_bit_cast(float, (268u - me) << 23);
      auto low = [&](float f, _Float16 h) { return (_Float16)(f * scale - (float)h); };
      typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
      f16x4 hi, lo;
#pragma unroll
      for (int i = 0; i < 4; ++i) hi[i] = half_of_nonzero(v[i] * scale, v[i]), lo[i] = low(v[i], hi[i]);
      *reinterpret_cast<f16x4 *>(x + half_off(4 * li)) = hi;
      *reinterpret_cast<f16x4 *>(x + half_off(4 * li) + 16) = lo;
      const _Float16 ph = half_of_nonzero(pv * scale, pv);
      *reinterpret_cast<_Float16 *>(x + half_off(DK + lp)) = ph;
      *reinterpret_cast<_Float16 *>(x + half_off(DK + lp) + 16) = low(pv, ph);
      if (lane == 0) rowU[er] = __builtin_bit_cast(float, (me - 14u) << 23);
    }
  };
  auto put_holding = [&](float *obs, int i) {
    const float v = (float)h[i] * d.s_hold;
    __builtin_nontemporal_store(v, &obs[(size_t)n * S + 1 + D + dd[i]]);
    O::store1(penv + O::off(dd[i]), v);
  };
  auto put_cash = [&](float *obs) {
    if (tl == 0) {
      const float v = cash * d.s_cash;
      __builtin_nontemporal_store(v, &obs[(size_t)n * S]);
      O::store1(penv + O::off(D), v);
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
      mu[i] = finish_out(((m[0] + m[PLANE]) + (m[2 * PLANE] + m[3 * PLANE])) * lu3[dd[i]], lb3[dd[i]], 1);
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
int hidden_bytes(int D) {
  const size_t trades = trade_lds(E, true, D) - (size_t)E * ((D + 3) & ~3) * 8;  // (the terms have a place of their own)
  return (int)((max(trades, (size_t)E * HP) + 15) & ~(size_t)15);
}

template <int E>
size_t lds_bytes(int D, int K) {
  using G = Geometry<E>;
  return (size_t)E * (half_pitch(f32_market_blocks(D, K)) + tile_pitch<false>(f32_portfolio_blocks(D))) + hidden_bytes<E>(D) +
         ((size_t)NM * G::PLANE + 2 * (2 * 256 + 32) + E) * 4 + (size_t)E * 32 * 8 + (size_t)NM * G::NL * 2048;
}

template <int E, int NH, int NP>
hipError_t launch_inst(hipStream_t st, const F32Args &a, size_t lds) {
  constexpr auto kern = rollout_f32_kernel<E, NH, NP>;
  const hipError_t e = allow_full_lds<kern>();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)(a.d.N / E)), dim3(NT), lds, st, a);
  return hipGetLastError();
}

template <int E, int NH, int NP>
hipError_t launch_geometry(hipStream_t st, F32Args a) {
  const EnvDims &d = a.d;
  a.market = f32_market_blocks(d.D, d.K), a.portfolio = f32_portfolio_blocks(d.D), a.hidden_bytes = hidden_bytes<E>(d.D);
  const size_t lds = lds_bytes<E>(d.D, d.K);
  if (d.N % E || a.envs_per_agent % E || d.D > 32 || lds > (size_t)kMaxLdsBytes) return hipErrorInvalidValue;
  constexpr int KIN = Geometry<E>::KIN;
  // Layer 1 in straight-line code, each block's inputs read a block ahead, for the blocks of 30 stocks x 8 indicators (257 to
  // 288 or 272 market columns).  us a step with numbers of blocks at run time and this: 16 envs, 1024 envs 6.64 and 6.57; 32
  // envs, 8192 14.4 and 14.2, 65536 of 64 agents 114 and 110.
  if ((d.D * d.K + d.D + KIN - 1) / KIN == NH && (d.D + KIN) / KIN == NP) return launch_inst<E, NH, NP>(st, a, lds);
  return launch_inst<E, 0, 0>(st, a, lds);
}

// 16 envs up to a workgroup for each of the 256 compute units; beyond, the weights streamed once for 32 envs are worth
// more (301 inputs, per step: 4096 envs 7.9 us against 11.8; 8192 in two rounds of 16 would be 15.8 against 14.2).
bool sixteen(int N) { return N <= 256 * 16; }

}  // namespace

size_t fused_f32_lds_bytes(const pr_config &c) {
  return sixteen(c.n_envs) ? lds_bytes<16>(c.n_stocks, c.n_ind) : lds_bytes<32>(c.n_stocks, c.n_ind);
}

hipError_t launch_rollout_fused_f32(hipStream_t st, const EnvDims &d, const EnvState &s, const float *price, const float *ind,
                                    const PackedNet &actor, int32_t envs_per_agent, int32_t T, const float *noise,
                                    const pr_buffers &out) {
  F32Args a;
  a.d = d, a.st = s, a.price = price, a.ind = ind, a.actor = actor, a.envs_per_agent = envs_per_agent, a.T = T;
  a.noise = noise, a.obs = out.obs, a.act_raw = out.act_raw, a.reward = out.reward, a.done = out.done, a.logp = out.logp;
  a.mu_out = out.mu, a.shares = out.shares;
  if (actor.bf16 || !actor.half_w[0] || actor.nkb[1] != 16 || actor.nct[0] != 8 || actor.nct[2] != 1) return hipErrorInvalidValue;
  return sixteen(d.N) ? launch_geometry<16, 9, 1>(st, a) : launch_geometry<32, 17, 2>(st, a);
}

}  // namespace pod
