// Rollout and value head of bf16 networks whose envs all read one shared market table (replay; 33 to 128 stocks).
//
// Nine tenths of an observation are a row of the table, and every env that
// stands on the row has the same ones.  What layer 1 makes of them,
//     P[row] = b1 + W1[indicators, prices] row            (fp32, as accumulated),
// is formed once per call and row instead of once per env and step; layer 1 of
// a step is then P[row] + W1[holdings, cash] (holdings, cash), one to nine
// k-blocks.  With that the policy's inputs fit in LDS next to the trades, and a
// workgroup keeps its envs on its compute unit for a whole rollout, as the
// persistent schedule does for fewer stocks.
// A rollout of 128 steps of 5000 envs x 100 stocks x 8 indicators over 16384
// rows, values and advantages included: 7.97 -> 3.31 ms (four launches a step
// 49.5 us -> 21 us; P of either network 30 us; value head 1.72 -> 0.6 ms).
// 8192 envs x 120 stocks, 32 steps 2.89 -> 1.49 ms, 512 x 60 0.74 -> 0.53, 16
// envs x 40, 64 steps 1.11 -> 0.67.  Calls of two steps are level or faster from
// 16 envs on; of one step only some: us without values over a table of 8000 rows, launches per step -> this (stocks x indicators)
//   envs          1            32            200           1000          2500          4000
//    40 x 2  17.3 -> 18.4  20.3 -> 19.5  21.0 -> 20.9  23.2 -> 24.0  29.9 -> 27.6  33.2 -> 32.1
//   100 x 8  21.6 -> 26.8  26.6 -> 28.4  30.2 -> 30.0  35.1 -> 37.2  44.4 -> 42.2  48.8 -> 51.9
//   128 x 4  21.1 -> 25.1  26.1 -> 26.8  28.3 -> 28.5  33.3 -> 34.5  41.7 -> 39.5  45.3 -> 46.9
// They are not sent back to those launches: layer 1's sums would have another
// order, and a rollout gives the same bits however it is cut into calls.
//
// Compiled with floating-point contraction off (pod_trade.h); the network code
// uses explicit fmaf.
#include "pod_internal.h"
#include "pod_tile.h"
#include "pod_trade.h"

namespace pod {
namespace {

using namespace tile;

constexpr int NW = 8, NT = NW * 64;
constexpr int kHidden = 512, kTiles = kHidden / 32, CTH = kTiles / NW;
constexpr int kPitch = kHidden + 16;  // floats per row of P (rows a multiple of 128 bytes apart fall on the same sets of the L1)
constexpr int kBlocks2 = kHidden / 16;
constexpr int PD = 8;                 // k-blocks of weights in flight
constexpr int HP = tile_pitch<true>(kBlocks2);

typedef f32x4 f32x4u __attribute__((aligned(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef f32x2 f32x2u __attribute__((aligned(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// A feature tile's sums of a row lie in P as one lane of the product holds them: 16 floats of half g = 0, then of half 1.
// Requests are 16 rows x 64 bytes (a quarter of the wavefront per 16 bytes), which the L1 serves four times as fast as the
// 32 rows x 32 bytes the accumulators' own layout would ask for; swaps between the lane quarters put them in order, either
// way: register i of quarter q <-> register q of quarter i.
__device__ inline void transpose_quarters(f32x4 (&v)[4]) {
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    uint32_t r[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float f = v[i][c];
      r[i] = __builtin_bit_cast(uint32_t, f);
    }
#pragma unroll
    for (int p = 0; p < 4; p += 2) {
      const auto s = __builtin_amdgcn_permlane16_swap(r[p], r[p + 1], false, false);
      r[p] = s[0], r[p + 1] = s[1];
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const auto s = __builtin_amdgcn_permlane32_swap(r[p], r[p + 2], false, false);
      r[p] = s[0], r[p + 2] = s[1];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t u = r[i];
      v[i][c] = __builtin_bit_cast(float, u);
    }
  }
}

__device__ inline void acc_from(f32x16 &acc, const f32x4 (&v)[4]) {
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[4 * j + i] = v[j][i];
}

// Table row of an env `t` steps after the cursor tau (an episode is the H rows from its start row).
__device__ inline int32_t row_after(int32_t tau, int32_t start, int32_t H, int64_t t) {
  const int64_t off = (int64_t)tau - start + t;
  return (int32_t)(off < H || tau - start >= H ? start + off : start + (off - H) % H);
}

// ------------------------------------------------------- market part of layer 1
struct MarketArgs {
  const float *price, *ind;  // [table rows][D], [table rows][D K]
  const u32x4 *W;            // market blocks [nkb][16][64], inputs [indicators | prices], each from a multiple of four on
  const float *b;            // b1
  float *P;                  // [rows][kPitch]
  int32_t rows, D, DK, nkb;
  float s_price, s_ind;
  // PAIRS: row r is what env r % N stands on r / N steps from now
  const int32_t *tau, *start;
  int32_t N, H, table_rows;
};

constexpr int kChunk = 8;  // k-blocks staged at a time
template <int I>
using Int = std::integral_constant<int, I>;

// 64 rows x 512 features per workgroup; the rows travel through two LDS buffers CKB k-blocks at a time, requested
// behind the chunk before.  A sum is one chain over the k-blocks whichever rows share a tile, so a row's P is the same number in
// any mode.  FEW: 128 features per workgroup, for launches of fewer than 64 tiles (a call of one step of 200
// envs x 100 stocks 72 -> 66 us).  FEWEST: 32 rows x 32 features per workgroup, one wavefront of which multiplies, up to a
// workgroup per compute unit: four workgroups draw 64 rows and all weights through four compute units (12 us of 900 market inputs, and
// 13 with requests as far ahead as here).  Calls of one step, 100 stocks x 8, 64 envs 34.1 -> 28.6 us, 400 36.4 -> 31.2, 600 37.2 -> 38.4
// (which stay with FEW); 128 x 4, 200 envs 32.2 -> 28.5.
enum Rows { MANY, FEW, FEWEST };
template <bool PAIRS, Rows MODE>
__global__ __launch_bounds__(NT, 2) void market_rows_kernel(MarketArgs a) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int CT = MODE == MANY ? CTH : 1, NBT = MODE == MANY ? 2 : 1, RD = MODE == FEWEST ? 8 : 4;
  constexpr int PC = MODE == FEWEST ? 4 : 1, RINGS = MODE == FEWEST ? 2 : 1;  // chunks of rows, and rings of weights, under way
  constexpr int CKB = kChunk, PITCH = tile_pitch<true>(CKB), GR = 4 * CKB, ROWS = MODE == FEWEST ? 32 : 64, NX = ROWS * GR / NT;
  const int row0 = blockIdx.x * ROWS, bt0 = MODE == FEW ? w >> 2 : 0;
  const int ct0 = MODE == MANY ? w * CT : MODE == FEW ? blockIdx.y * 4 + (w & 3) : blockIdx.y;
  const bool multiplies = MODE != FEWEST || w == 0;
  const int DK = a.DK, DK4 = (DK + 3) & ~3, nch = (a.nkb + CKB - 1) / CKB;

  // A thread stages four columns of NX rows.  Every request is made and lies inside its row: a group that reaches past the end
  // of the indicators or of the prices is read as the four numbers that end there and shifted.  (With branches around the
  // requests 190 registers spilled.)
  int row[NX];
#pragma unroll
  for (int i = 0; i < NX; ++i) {
    int r = min(row0 + tid / GR + NT / GR * i, a.rows - 1);
    if (PAIRS) {
      const int n = r % a.N;
      r = row_after(a.tau[n], a.start[n], a.H, r / a.N);
    }
    row[i] = min(max(r, 0), a.table_rows - 1);
  }
  f32x4 pre[PC][NX];
  auto fetch = [&](int ch, f32x4(&pre)[NX]) {
    ch = min(ch, nch - 1);
    int l = threadIdx.x;
    asm volatile("" : "+v"(l));
    const int c = ch * (16 * CKB) + 4 * (l & (GR - 1));
    const bool is_ind = c < DK4;
    const float *base = is_ind ? a.ind + min(c, DK - 4) : a.price + min(c - DK4, a.D - 4);
    const int64_t pitch = is_ind ? DK : a.D;
#pragma unroll
    for (int i = 0; i < NX; ++i) pre[i] = *reinterpret_cast<const f32x4u *>(base + row[i] * pitch);
  };
  auto stash = [&](int ch, const f32x4(&pre)[NX]) {
    int l = threadIdx.x;
    asm volatile("" : "+v"(l));
    const int c = ch * (16 * CKB) + 4 * (l & (GR - 1));
    const bool is_ind = c < DK4;
    const float scale = is_ind ? a.s_ind : a.s_price;
    const int back = is_ind ? c - min(c, DK - 4) : c - DK4 - min(c - DK4, a.D - 4);
    const bool ends = __ballot(back != 0) != 0;
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      f32x4 v = pre[i] * scale;
      if (ends) {
        if (back & 1) v = f32x4{v[1], v[2], v[3], 0.0f};
        if (back & 2) v = f32x4{v[2], v[3], 0.0f, 0.0f};
        if (back >= 4) v = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      }
      Op<true>::store4(lds + (ch & 1) * (ROWS * PITCH) + (l / GR + NT / GR * i) * PITCH + 8 * (l & (GR - 1)), v[0], v[1], v[2], v[3]);
    }
  };

  const u32x4 *wp[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) wp[c] = a.W + (size_t)(ct0 + c) * 64 + lane;
  u32x4 ring[RINGS][RD][CT];
#pragma unroll
  for (int j = 0; j < PC; ++j) {
    fetch(j, pre[j]);
    if (j < RINGS && multiplies) {
#pragma unroll
      for (int s = 0; s < RD; ++s)
#pragma unroll
        for (int c = 0; c < CT; ++c) ring[j % RINGS][s][c] = wp[c][(size_t)min(j * RD + s, a.nkb - 1) * kTiles * 64];
    }
  }
  f32x16 acc[CT][NBT];
  bias_acc<CT, NBT>(acc, a.b, ct0, lane);
  const int nfull = a.nkb / CKB;
#pragma unroll
  for (int i = 0; i < NX; ++i) asm volatile("" : "+v"(pre[0][i]));  // (arrived: the loop's waits are for its own requests)
  auto chunk = [&](int ch, auto place) {  // place: ch % PC
    constexpr int j = decltype(place)::value;
    unsigned char *x = lds + (ch & 1) * (ROWS * PITCH);
    stash(ch, pre[j]);
    __syncthreads();  // chunk ch complete; everybody is done with the buffer chunk ch + 1 goes into
    fetch(ch + PC, pre[j]);
    asm volatile("" ::: "memory");  // (requested here: behind the weights they would be waited for with them)
    __builtin_amdgcn_sched_barrier(0);
    if (multiplies)
      mma_chunk<CT, NBT, RD, CKB, RINGS * RD>(acc, ring[j % RINGS], x + bt0 * (32 * PITCH), PITCH, ch * CKB, a.nkb, wp, kTiles, lane);
  };
  auto last = [&](auto place) {
    constexpr int j = decltype(place)::value;
    stash(nfull, pre[j]);
    __syncthreads();
    if (multiplies)
      mma_layer_range<true, CT, NBT, RD>(acc, ring[j % RINGS], lds + (nfull & 1) * (ROWS * PITCH), PITCH, nfull * CKB, a.nkb, a.nkb, a.W, kTiles,
                                         ct0, bt0, lane);
  };
  int ch = 0;
  if constexpr (PC == 4) {
    for (; ch + 4 <= nfull; ch += 4) chunk(ch, Int<0>{}), chunk(ch + 1, Int<1>{}), chunk(ch + 2, Int<2>{}), chunk(ch + 3, Int<3>{});
    if (ch < nfull) chunk(ch, Int<0>{});
    if (ch + 1 < nfull) chunk(ch + 1, Int<1>{});
    if (ch + 2 < nfull) chunk(ch + 2, Int<2>{});
    if (nfull < nch) {
      switch (nfull & 3) {
        case 0: last(Int<0>{}); break;
        case 1: last(Int<1>{}); break;
        case 2: last(Int<2>{}); break;
        case 3: last(Int<3>{}); break;
      }
    }
  } else {
    for (; ch < nfull; ++ch) chunk(ch, Int<0>{});
    if (nfull < nch) last(Int<0>{});
  }
  if (!multiplies) return;
#pragma unroll
  for (int c = 0; c < CT; ++c)
#pragma unroll
    for (int t = 0; t < NBT; ++t) {
      f32x4 v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = f32x4{acc[c][t][4 * j], acc[c][t][4 * j + 1], acc[c][t][4 * j + 2], acc[c][t][4 * j + 3]};
      transpose_quarters(v);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = row0 + 32 * (bt0 + t) + 16 * (i & 1) + (lane & 15);
        if (r < a.rows)
          *reinterpret_cast<f32x4 *>(a.P + (size_t)r * kPitch + (ct0 + c) * 32 + 16 * (i >> 1) + 4 * (lane >> 4)) = v[i];
      }
    }
}

// ------------------------------------------------------------------- rollout
struct TableArgs {
  EnvDims d;
  EnvState st;
  const float *price, *ind;
  const float *P;
  const u32x4 *Wp, *W2, *W3;  // [kb][16][64] (inputs [holdings | 0 | cash]), [32][16][64], [32][nct3][64]
  const float *b2, *b3;
  int32_t *tau0;              // [N] cursors at the start of the call, or null
  int32_t per;                // envs per workgroup, at most E
  int32_t nct3;
  int32_t pairs;              // P is indexed by (step, env) instead of by table row
  int32_t p_rows;             // rows of P
  int32_t T;
  int32_t first;              // the first observation is written too
  const float *noise;
  float *obs, *act_raw, *reward;
  uint8_t *done;
  float *logp, *mu;           // opt
  int32_t *shares;            // opt
};

template <int E, int KBP>
struct TableGeo {
  static constexpr int TPE = NT / E;
  static constexpr int DMAX = 16 * KBP - 1 < 128 ? 16 * KBP - 1 : 128;
  static constexpr int ND = (DMAX + TPE - 1) / TPE;
  static constexpr int XP = tile_pitch<true>(KBP);
  // two hidden tiles; the planes of output sums lie over the first: four parts of 64 columns or two of 128
  static constexpr int H2 = E * 4 * 68 * 4;
  static constexpr size_t net = (size_t)H2 + E * HP;
  static_assert(H2 >= E * HP && H2 >= E * 2 * 132 * 4, "");
  static size_t lds(int D) {
    const size_t tr = trade_lds(E, false, D);
    return (size_t)E * XP + (size_t)(kHidden + 128) * 4 + (size_t)2 * E * 4 + (tr > net ? tr : net);
  }
};

// A workgroup steps `per` envs (E slots: one 32-column operand, half of it empty with E = 16) for T steps.  Per step:
// layer 1's portfolio blocks on top of P, layer 2, layer 3 with the inputs split over wavefronts, then the trades of
// pod_trade.h.  The weights (0.73 MB with 100 stocks) stream from L2 through a ring of 8 k-blocks in registers that runs on
// across the layers and is primed for the next step, like the next rows of P, beside the trades.  The wavefronts the trades
// leave over move the market part of the next observation.
// What bounds a step of 20 envs x 100 stocks (time stamps, thousands of cycles of 46): layer 1 4, layer 2 11 (52 bytes of
// weights a cycle and compute unit, of 64), layer 3 2, sampling 3.5, sizing 4, ledger 7, requests and bookings 9; without
// the moves it would take 4 us less.
template <int E, int KBP>
__global__ __launch_bounds__(NT, 2) void rollout_table_kernel(TableArgs a) {
  using G = TableGeo<E, KBP>;
  constexpr int TPE = G::TPE, ND = G::ND, XP = G::XP;
  using Tr = Trade<E, ND, false, kEnvThreads, true>;
  extern __shared__ __align__(16) unsigned char lds[];
  const EnvDims &d = a.d;
  const int D = d.D, DK = D * d.K, S = d.S, NG = DK / 4;
  const size_t N = (size_t)d.N;
  unsigned char *ldsX = lds;
  float *ldsB = reinterpret_cast<float *>(ldsX + E * XP);            // b2 | b3
  int32_t *s_row = reinterpret_cast<int32_t *>(ldsB + kHidden + 128);  // table row of the next observation
  int32_t *s_prow = s_row + E;                                       // and its row of P
  unsigned char *ldsT = reinterpret_cast<unsigned char *>(s_prow + E);
  unsigned char *ldsH = ldsT, *ldsH2 = ldsT + G::H2;
  float *planes = reinterpret_cast<float *>(ldsH);                   // [parts][E][MP], once the first hidden tile is read
  Tr trade(ldsT, D);

  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n0 = blockIdx.x * a.per, last = min(a.per, d.N - n0) - 1;  // (envs beyond the last one follow it and write nothing)
  const int ct0 = w * CTH, traders = min(NW, (a.per * TPE + 63) / 64);
  // The thread's env and its first stock.  (Formed anew in every step from an opaque thread index: what follows from them would
  // be kept in registers across the steps.)
  struct Own {
    int e, tl, n;
    bool live;
  };
  auto own = [&]() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    const int e = t / TPE;
    return Own{e, t & (TPE - 1), n0 + min(e, last), e <= last};
  };

  for (int i = tid; i < E * XP / 4; i += NT) reinterpret_cast<uint32_t *>(ldsX)[i] = 0u;
  for (int i = tid; i < kHidden; i += NT) ldsB[i] = a.b2[i];
  if (tid < 32 * a.nct3) ldsB[kHidden + tid] = a.b3[tid];

  // -- state
  const Own o0 = own();
  int32_t tau = a.st.tau[o0.n];
  const int32_t start = a.st.start[o0.n];
  float cash = a.st.cash[o0.n];
  int32_t h[ND];
  float pn[ND], eps[ND], pv[ND];
  double ep_ret = a.st.ep_ret[o0.n], ep_sum = a.st.ep_sum[o0.n], ep_sqsum = a.st.ep_sqsum[o0.n];
  int32_t ep_cnt = a.st.ep_cnt[o0.n];
  if (a.tau0 && o0.live && o0.tl == 0) a.tau0[o0.n] = tau;

  // noise and prices of step t at cursor tau
  auto request_step = [&](int t, int32_t tau_t) {
    const Own m = own();
    const RowInfo r = rows_of(d, tau_t, start, m.n);
    const size_t g = ((size_t)t * N + m.n) * D;
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      const int dd = min(m.tl + TPE * i, D - 1);
      eps[i] = __builtin_nontemporal_load(a.noise + g + dd);
      pv[i] = a.price[(size_t)r.row_val * D + dd];
    }
  };
  // layer-1 sums of the market part: 16 rows x 64 bytes a request
  f32x4 pr[CTH][4];
  auto request_market_sums = [&]() {
    int l = threadIdx.x & 63;
    asm volatile("" : "+v"(l));
#pragma unroll
    for (int rh = 0; rh < E / 16; ++rh) {
      const float *p = a.P + (size_t)s_prow[16 * rh + (l & 15)] * kPitch + ct0 * 32 + 4 * (l >> 4);
#pragma unroll
      for (int c = 0; c < CTH; ++c)
#pragma unroll
        for (int g = 0; g < 2; ++g) pr[c][2 * g + rh] = *reinterpret_cast<const f32x4 *>(p + 32 * c + 16 * g);
    }
    if (E == 16) {
#pragma unroll
      for (int c = 0; c < CTH; ++c) pr[c][1] = pr[c][0], pr[c][3] = pr[c][2];
    }
  };
  // the weights of a step in the order they are used: KBP blocks of layer 1, 32 of layer 2, pairs of blocks of layer 3
  u32x4 ring[PD][CTH];
  const int nct3 = a.nct3, n3 = nct3 == 2 ? 2 : 4, ct3 = min(w % n3, nct3 - 1), part3 = w / n3;
  const int MP = n3 == 2 ? 68 : 132;  // row pitch of a plane
  const u32x4 *Wp = a.Wp + ct0 * 64, *W2 = a.W2 + ct0 * 64;
  const u32x4 *W3 = a.W3 + (part3 * (n3 == 2 ? 8 : 16) * nct3 + ct3) * 64;
  // (a lane's offset in bytes: with block offsets added to the uniform address 190 scalar registers spilled)
  auto block = [&](const u32x4 *W, uint32_t blocks, int l) {
    return *reinterpret_cast<const u32x4 *>(reinterpret_cast<const unsigned char *>(W) + (uint32_t)(blocks * 1024u + (uint32_t)l * 16u));
  };
  auto request_weights = [&](int q, int l) {  // q is a compile-time number
    u32x4(&slot)[CTH] = ring[q % PD];
#pragma unroll
    for (int c = 0; c < CTH; ++c) {
      if (q < KBP) slot[c] = block(Wp, q * kTiles + c, l);
      else if (q < KBP + kBlocks2) slot[c] = block(W2, (q - KBP) * kTiles + c, l);
      else if (q < KBP + kBlocks2 + 4 || n3 == 4) slot[c] = block(W3, (2 * (q - KBP - kBlocks2) + c) * nct3, l);
    }
  };

  // (streamed past the L2, which the weights stay in)
  auto put = [](float *p, f32x4 v) { __builtin_nontemporal_store(v, reinterpret_cast<f32x4u *>(p)); };
  // Market part of an observation: a wavefront moves rows first, first + stride, ... of the workgroup's, R at a time, 64
  // groups of four indicators a request.
  auto move_market = [&](float *obs_row0, int first, int stride, auto rows) {
    constexpr int R = decltype(rows)::value;
    int l = threadIdx.x & 63;
    asm volatile("" : "+v"(l));
    for (int r = first; r <= last; r += R * stride) {
      const float *src[R], *ps[R];
      float *o[R];
      bool is[R];
#pragma unroll
      for (int k = 0; k < R; ++k) {
        const int er = min(r + k * stride, last);
        is[k] = r + k * stride <= last;
        const size_t row = (size_t)__builtin_amdgcn_readfirstlane(s_row[er]);
        src[k] = a.ind + row * DK, ps[k] = a.price + row * D;
        o[k] = obs_row0 + (size_t)(n0 + er) * S + 1;
      }
      float p[R][2];
#pragma unroll
      for (int k = 0; k < R; ++k)
#pragma unroll
        for (int j = 0; j < 2; ++j) p[k][j] = ps[k][min(l + 64 * j, D - 1)];
      for (int g0 = l; g0 < NG; g0 += 4 * 64) {
        f32x4 v[R][4];
#pragma unroll
        for (int k = 0; k < R; ++k)
#pragma unroll
          for (int j = 0; j < 4; ++j) v[k][j] = *reinterpret_cast<const f32x4u *>(src[k] + 4 * min(g0 + 64 * j, NG - 1));
#pragma unroll
        for (int k = 0; k < R; ++k)
          if (is[k])
#pragma unroll
            for (int j = 0; j < 4; ++j) put(o[k] + 2 * D + 4 * min(g0 + 64 * j, NG - 1), v[k][j] * d.s_ind);
      }
#pragma unroll
      for (int k = 0; k < R; ++k)
        if (is[k]) {
#pragma unroll
          for (int j = 0; j < 2; ++j) o[k][min(l + 64 * j, D - 1)] = p[k][j] * d.s_price;
          if (l < (DK & 3)) o[k][2 * D + 4 * NG + l] = src[k][4 * NG + l] * d.s_ind;
        }
    }
  };
  using Two = std::integral_constant<int, 2>;
  auto put_holding = [&](float *o, int e, int dd, int32_t x) {
    const float v = (float)x * d.s_hold;
    if (o) o[1 + D + dd] = v;
    Op<true>::store1(ldsX + e * XP + 2 * dd, v);
  };
  auto put_cash = [&](float *o, int e, float c) {
    const float v = c * d.s_cash;
    if (o) o[0] = v;
    Op<true>::store1(ldsX + e * XP + 2 * (16 * KBP - 1), v);
  };

  // -- the first observation
  if (o0.tl == 0) {
    s_row[o0.e] = tau;
    s_prow[o0.e] = min(max(a.pairs ? o0.n : tau, 0), a.p_rows - 1);
  }
  __syncthreads();
  {
    float *o = a.first && o0.live ? a.obs + (size_t)o0.n * S : nullptr;
    request_step(0, tau);
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      const int dd = o0.tl + TPE * i, dc = min(dd, D - 1);
      pn[i] = a.price[(size_t)tau * D + dc];
      h[i] = a.st.h[(size_t)o0.n * D + dc];
      if (dd < D) {
        put_holding(o, o0.e, dd, h[i]);
      }
    }
    if (o0.tl == 0) put_cash(o, o0.e, cash);
    if (a.first) move_market(a.obs, w, NW, Two{});
  }
  request_market_sums();
#pragma unroll
  for (int q = 0; q < PD; ++q) request_weights(q, lane);

  for (int t = 0; t < a.T; ++t) {
    __syncthreads();  // the observation's portfolio part is complete
    // (opaque per step: the addresses of the weight blocks are formed again instead of being kept across the loop)
    int l = lane;
    asm volatile("" : "+v"(l));
    asm volatile("" : "+s"(Wp), "+s"(W2), "+s"(W3));
    const int brow = l & (E - 1), half = l >> 5;
    const bool row_lane = (l & 31) < E;
    if (w < traders) {
      const Own m = own();
      const RowInfo r = rows_of(d, tau, start, m.n);
      if (m.tl == 0) {
        s_row[m.e] = r.row_obs;
        s_prow[m.e] = min(max(a.pairs ? min(t + 1, a.T - 1) * d.N + m.n : r.row_obs, 0), a.p_rows - 1);
      }
    }
    // -- layer 1
    f32x16 acc[CTH][1];
#pragma unroll
    for (int c = 0; c < CTH; ++c) {
      transpose_quarters(pr[c]);
      acc_from(acc[c][0], pr[c]);
    }
    {
      const unsigned char *x = ldsX + brow * XP + 16 * half;
      u32x4 xn = *reinterpret_cast<const u32x4 *>(x);
#pragma unroll
      for (int i = 0; i < KBP; ++i) {
        const u32x4 xv = xn;
        if (i + 1 < KBP) xn = *reinterpret_cast<const u32x4 *>(x + 32 * (i + 1));
#pragma unroll
        for (int c = 0; c < CTH; ++c) Op<true>::mma(ring[i % PD][c], xv, acc[c][0]);
        request_weights(i + PD, l);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    auto put_hidden = [&](unsigned char *H) {
#pragma unroll
      for (int c = 0; c < CTH; ++c) {
        tanh_in_place<1>(acc[c]);
        if (row_lane) {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            Op<true>::store4(H + brow * HP + ((ct0 + c) * 32 + 8 * j + 4 * half) * 2, acc[c][0][4 * j], acc[c][0][4 * j + 1],
                             acc[c][0][4 * j + 2], acc[c][0][4 * j + 3]);
        }
      }
    };
    put_hidden(ldsH);
    __syncthreads();
    // -- layer 2
    bias_acc<CTH, 1>(acc, ldsB, ct0, l);
    {
      const unsigned char *x = ldsH + brow * HP + 16 * half;
      u32x4 xn = *reinterpret_cast<const u32x4 *>(x);
#pragma unroll
      for (int i = 0; i < kBlocks2; ++i) {
        const u32x4 xv = xn;
        if (i + 1 < kBlocks2) xn = *reinterpret_cast<const u32x4 *>(x + 32 * (i + 1));
#pragma unroll
        for (int c = 0; c < CTH; ++c) Op<true>::mma(ring[(KBP + i) % PD][c], xv, acc[c][0]);
        request_weights(KBP + i + PD, l);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    put_hidden(ldsH2);
    __syncthreads();
    // -- layer 3: its blocks are in the ring
    {
      f32x16 o3;
#pragma unroll
      for (int i = 0; i < 16; ++i) o3[i] = 0.0f;
      const int kb0 = part3 * (n3 == 2 ? 8 : 16);
      const unsigned char *x = ldsH2 + brow * HP + 16 * half + 32 * kb0;
      auto blocks = [&](int q0) {
        u32x4 xv[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) xv[i] = *reinterpret_cast<const u32x4 *>(x + 32 * (8 * q0 + i));
#pragma unroll
        for (int i = 0; i < 8; ++i) Op<true>::mma(ring[(KBP + kBlocks2 + 4 * q0 + i / 2) % PD][i % 2], xv[i], o3);
      };
      blocks(0);
      if (n3 == 4) blocks(1);
      if (row_lane && w % n3 < nct3) {
        float *p = planes + (part3 * E + brow) * MP + ct3 * 32 + 4 * half;
#pragma unroll
        for (int j = 0; j < 4; ++j) *reinterpret_cast<f32x4 *>(p + 8 * j) = f32x4{o3[4 * j], o3[4 * j + 1], o3[4 * j + 2], o3[4 * j + 3]};
      }
    }
    __syncthreads();
    // The trades take the first `traders` wavefronts; those left over, if any, move the market part of the next observation
    // and sum the noise meanwhile.
    float *obs_next = a.obs + (size_t)(t + 1) * N * S;
    if (w < traders) {
      const Own m = own();
      const int e = m.e, tl = m.tl, n = m.n;
      const bool live = m.live;
      const RowInfo ri = rows_of(d, tau, start, n);
      trade.me = e * TPE + tl;
      float a_raw[ND];
      const size_t g0 = ((size_t)t * N + n) * D;
#pragma unroll
      for (int i = 0; i < ND; ++i) {
        const int dd = min(tl + TPE * i, D - 1);
        const float *p = planes + e * MP + dd;
        float z = p[0] + p[E * MP];
        if (n3 == 2) z = z + p[2 * E * MP], z = z + p[3 * E * MP];
        const float mu = finish_out(z, ldsB[kHidden + dd], 1);
        a_raw[i] = mu + d.sigma * eps[i];  // two roundings (contraction is off)
        if (live && tl + TPE * i < D) {
          a.act_raw[g0 + dd] = a_raw[i];
          if (a.mu) a.mu[g0 + dd] = mu;
        }
      }
      __syncthreads();  // the planes are read: the trades' scratch lies over them
      float *o = obs_next + (size_t)n * S;
      int32_t q[ND];
      float e2;
      double r;
      trade.run(
          d, live, a_raw, eps, pn, Tr::unit_of(d, pn), pv, h, q, cash, r, e2, a.logp != nullptr && traders == NW,
          [&]() {
            if (traders == NW) move_market(obs_next, w, NW, Two{});
          },
          [&]() {
            // (requested in front of the step's last stores: a wavefront's memory operations complete in order)
            request_market_sums();
#pragma unroll
            for (int q = 0; q < PD; ++q) request_weights(q, l);
          },
          [&](int i) {
            const int dd = tl + TPE * i;
            if (ri.done) h[i] = 0;
            put_holding(o, e, dd, h[i]);
            if (a.shares) a.shares[g0 + dd] = q[i];
          });
      ep_ret += r;
      if (ri.done) {
        ep_sum += ep_ret;
        ep_sqsum += ep_ret * ep_ret;
        ep_cnt += 1;
        ep_ret = 0.0;
        cash = d.cash0;
      }
      if (live && tl == 0) {
        put_cash(o, e, cash);
        a.reward[(size_t)t * N + n] = (float)r;
        a.done[(size_t)t * N + n] = (uint8_t)ri.done;
        if (a.logp && traders == NW) a.logp[(size_t)t * N + n] = fmaf(-0.5f, e2, d.logp_const);
      }
      // prices of the next observation: those the account is valued at, but for an episode's end
#pragma unroll
      for (int i = 0; i < ND; ++i) pn[i] = ri.done ? a.price[(size_t)ri.row_obs * D + min(tl + TPE * i, D - 1)] : pv[i];
      tau = ri.done ? start : tau + 1;
      request_step(min(t + 1, a.T - 1), tau);
    } else {
      __syncthreads();
      request_market_sums();
#pragma unroll
      for (int q = 0; q < PD; ++q) request_weights(q, l);
      move_market(obs_next, w - traders, NW - traders, Two{});
      if (w == NW - 1 && a.logp && l <= last) {
        // squares summed in stock order (a lane per env)
        const float *x = a.noise + ((size_t)t * N + n0 + l) * D;
        float e2 = 0.0f;
#pragma unroll 16
        for (int i = 0; i < D; ++i) {
          const float v = x[i] * x[i];
          e2 = e2 + v;
        }
        a.logp[(size_t)t * N + n0 + l] = fmaf(-0.5f, e2, d.logp_const);
      }
    }
  }

  const Own m = own();
  const int n = m.n;
#pragma unroll
  for (int i = 0; i < ND; ++i) {
    const int dd = m.tl + TPE * i;
    if (m.live && dd < D) a.st.h[(size_t)n * D + dd] = h[i];
  }
  if (m.live && m.tl == 0) {
    a.st.tau[n] = tau;
    a.st.cash[n] = cash;
    a.st.ep_ret[n] = ep_ret;
    a.st.ep_sum[n] = ep_sum;
    a.st.ep_sqsum[n] = ep_sqsum;
    a.st.ep_cnt[n] = ep_cnt;
  }
}

// ---------------------------------------------------------------- value head
struct ValueTableArgs {
  EnvDims d;
  const float *obs;           // [rows][S]
  int64_t rows;               // (T + 1) N
  const float *P;             // by table row
  int32_t p_rows;
  const int32_t *tau0, *start;
  const u32x4 *Wp, *W2;
  const __bf16 *w3;           // packed blocks of the output layer
  const float *b2, *b3;
  float *Y;
};

template <int KBP>
__global__ __launch_bounds__(NT, 2) void value_table_kernel(ValueTableArgs a) {
  constexpr int NBT = 2, XP = tile_pitch<true>(KBP), RPW = 64 / NW;
  constexpr int Q = KBP + kBlocks2;  // k-blocks of a tile; the ring runs on from one tile to the next
  extern __shared__ __align__(16) unsigned char lds[];
  unsigned char *ldsX = lds, *ldsH = ldsX + 64 * XP;
  float *ldsB = reinterpret_cast<float *>(ldsH + 64 * HP);
  float *ldsPart = ldsB + kHidden;                             // [2 NW][64]
  __bf16 *ldsW3 = reinterpret_cast<__bf16 *>(ldsPart + 2 * NW * 64);
  int32_t *s_prow = reinterpret_cast<int32_t *>(ldsW3 + kHidden);  // [64] rows of P of the next tile
  const EnvDims &d = a.d;
  const int D = d.D, S = d.S;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), ct0 = w * CTH;
  const int64_t ntiles = (a.rows + 63) / 64;

  auto find_rows = [&](int64_t tile) {  // (one wavefront)
    const int64_t r = min(tile * 64 + lane, a.rows - 1);
    const int64_t t = r / d.N;
    const int n = (int)(r - t * d.N);
    s_prow[lane] = min(max(row_after(a.tau0[n], a.start[n], d.H, t), 0), a.p_rows - 1);
  };
  f32x4 pr[CTH][NBT][4];
  auto request_market_sums = [&]() {
    int l = threadIdx.x & 63;
    asm volatile("" : "+v"(l));
#pragma unroll
    for (int t = 0; t < NBT; ++t)
#pragma unroll
      for (int rh = 0; rh < 2; ++rh) {
        const float *p = a.P + (size_t)s_prow[32 * t + 16 * rh + (l & 15)] * kPitch + ct0 * 32 + 4 * (l >> 4);
#pragma unroll
        for (int c = 0; c < CTH; ++c)
#pragma unroll
          for (int g = 0; g < 2; ++g) pr[c][t][2 * g + rh] = *reinterpret_cast<const f32x4 *>(p + 32 * c + 16 * g);
      }
  };
  // holdings and cash of rows 8 w .. 8 w + 7: two holdings a lane, the cash in the last column
  constexpr int last_col = 16 * KBP - 1;
  f32x2 xr[RPW];
  f32x2 x9[KBP > 8 ? RPW : 1];
  float cash;
  auto request_rows = [&](int64_t tile) {
    int l = threadIdx.x & 63;
    asm volatile("" : "+v"(l));
    const int64_t r0 = tile * 64 + RPW * w;
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
      const float *o = a.obs + min(r0 + i, a.rows - 1) * S + 1 + D;
      xr[i] = *reinterpret_cast<const f32x2u *>(o + min(2 * l, D - 1));
      if (KBP > 8) x9[i] = *reinterpret_cast<const f32x2u *>(o + min(128 + 2 * l, D - 1));
    }
    cash = a.obs[min(r0 + (l & 7), a.rows - 1) * S];
  };
  auto put_rows = [&]() {
    int l = threadIdx.x & 63;
    asm volatile("" : "+v"(l));
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
      const float c = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, cash), i));
      auto put = [&](int col, f32x2 v) {
        const float v0 = col < D ? v[0] : 0.0f, v1 = col + 1 < D ? v[1] : col + 1 == last_col ? c : 0.0f;
        if (col < 16 * KBP) *reinterpret_cast<bf16x2 *>(ldsX + (RPW * w + i) * XP + 2 * col) = bf16x2{(__bf16)v0, (__bf16)v1};
      };
      put(2 * l, xr[i]);
      if (KBP > 8) put(128 + 2 * l, x9[i]);
    }
  };
  u32x4 ring[4][CTH];
  auto request_weights = [&](int slot, int q, int l) {  // slot and q are compile-time numbers
#pragma unroll
    for (int c = 0; c < CTH; ++c)
      ring[slot][c] = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const unsigned char *>((q < KBP ? a.Wp : a.W2) + ct0 * 64) +
                                                       (uint32_t)(((q < KBP ? q : q - KBP) * kTiles + c) * 1024u + (uint32_t)l * 16u));
  };

  for (int i = tid; i < kHidden; i += NT) {
    ldsB[i] = a.b2[i];
    // output weights of feature 0 out of the packed blocks: k = 16 kb + 8 g + e sits in lane 32 g
    ldsW3[i] = a.w3[((size_t)(i >> 4) * 64 + 32 * ((i >> 3) & 1)) * 8 + (i & 7)];
  }
  const float b3 = a.b3[0];
  int64_t tile = blockIdx.x;
  if (w == 0) find_rows(tile);
  request_rows(tile);
  put_rows();
  __syncthreads();
  request_market_sums();
#pragma unroll
  for (int q = 0; q < 4; ++q) request_weights(q, q, lane);

  for (; tile < ntiles; tile += gridDim.x) {
    const int64_t next = min(tile + gridDim.x, ntiles - 1);
    int l = lane;
    asm volatile("" : "+v"(l));
    const int brow = l & 31, half = l >> 5;
    f32x16 acc[CTH][NBT];
#pragma unroll
    for (int c = 0; c < CTH; ++c)
#pragma unroll
      for (int t = 0; t < NBT; ++t) {
        transpose_quarters(pr[c][t]);
        acc_from(acc[c][t], pr[c][t]);
      }
    auto steps = [&](const unsigned char *x, int pitch, auto q0c, auto countc) {
      constexpr int q0 = decltype(q0c)::value, count = decltype(countc)::value;
#pragma unroll
      for (int i = 0; i < count; ++i) {
        u32x4 xv[NBT];
#pragma unroll
        for (int t = 0; t < NBT; ++t) xv[t] = *reinterpret_cast<const u32x4 *>(x + t * 32 * pitch + 32 * i);
#pragma unroll
        for (int c = 0; c < CTH; ++c)
#pragma unroll
          for (int t = 0; t < NBT; ++t) Op<true>::mma(ring[(q0 + i) % 4][c], xv[t], acc[c][t]);
        // (the next tile's first blocks go where it looks for them, once this tile's last use of those registers is past)
        if (q0 + i + 4 < Q) request_weights((q0 + i) % 4, q0 + i + 4, l);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    steps(ldsX + brow * XP + 16 * half, XP, std::integral_constant<int, 0>{}, std::integral_constant<int, KBP>{});
    epilogue_hidden_biased<CTH, NBT>(acc, ldsH, HP, ct0, 0, l);
    if (w == 0) find_rows(next);  // (read behind the barrier)
    __syncthreads();
    bias_acc<CTH, NBT>(acc, ldsB, ct0, l);
    steps(ldsH + brow * HP + 16 * half, HP, std::integral_constant<int, KBP>{}, std::integral_constant<int, kBlocks2>{});
#pragma unroll
    for (int q = 0; q < 4; ++q) request_weights(q, q, l);
    request_rows(next);
    request_market_sums();
    float part[NBT][4];
#pragma unroll
    for (int t = 0; t < NBT; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) part[t][j] = 0.0f;
#pragma unroll
    for (int c = 0; c < CTH; ++c) {
      tanh_in_place<NBT>(acc[c]);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const u32x2 wv = *reinterpret_cast<const u32x2 *>(ldsW3 + (ct0 + c) * 32 + 8 * j + 4 * half);
        const uint32_t wlo = wv[0], whi = wv[1];
        const bf16x2 w01 = __builtin_bit_cast(bf16x2, wlo), w23 = __builtin_bit_cast(bf16x2, whi);
#pragma unroll
        for (int t = 0; t < NBT; ++t) {
          const bf16x2 h01 = {(__bf16)acc[c][t][4 * j], (__bf16)acc[c][t][4 * j + 1]};
          const bf16x2 h23 = {(__bf16)acc[c][t][4 * j + 2], (__bf16)acc[c][t][4 * j + 3]};
          part[t][j] = __builtin_amdgcn_fdot2_f32_bf16(h01, w01, part[t][j], false);
          part[t][j] = __builtin_amdgcn_fdot2_f32_bf16(h23, w23, part[t][j], false);
        }
      }
    }
#pragma unroll
    for (int t = 0; t < NBT; ++t) ldsPart[(2 * w + half) * 64 + 32 * t + brow] = (part[t][0] + part[t][1]) + (part[t][2] + part[t][3]);
    put_rows();  // (layer 1 of this tile is past: the barrier above)
    __syncthreads();
    if (w == 0 && tile * 64 + lane < a.rows) {
      float y = b3;
#pragma unroll
      for (int p = 0; p < 2 * NW; ++p) y += ldsPart[p * 64 + lane];
      a.Y[tile * 64 + lane] = y;
    }
  }
}

// k-blocks of the portfolio part: the stocks, and the cash in the last column
int portfolio_blocks(int D) { return (D + 16) / 16; }

template <class Launch>
hipError_t with_blocks(int D, Launch launch) {
  switch (portfolio_blocks(D)) {
    case 3: return launch(std::integral_constant<int, 3>{});
    case 4: return launch(std::integral_constant<int, 4>{});
    case 5: return launch(std::integral_constant<int, 5>{});
    case 6: return launch(std::integral_constant<int, 6>{});
    case 7: return launch(std::integral_constant<int, 7>{});
    case 8: return launch(std::integral_constant<int, 8>{});
    case 9: return launch(std::integral_constant<int, 9>{});
  }
  return hipErrorInvalidValue;
}

template <int E, int KBP>
hipError_t launch_rollout_inst(hipStream_t st, const TableArgs &a) {
  constexpr auto kern = rollout_table_kernel<E, KBP>;
  const hipError_t err = allow_full_lds<kern>();
  if (err != hipSuccess) return err;
  const size_t lds = TableGeo<E, KBP>::lds(a.d.D);
  hipLaunchKernelGGL(kern, dim3((unsigned)((a.d.N + a.per - 1) / a.per)), dim3(NT), lds, st, a);
  return hipGetLastError();
}

template <int KBP>
hipError_t launch_rollout_blocks(hipStream_t st, const TableArgs &a) {
  return a.per <= 16 ? launch_rollout_inst<16, KBP>(st, a) : launch_rollout_inst<32, KBP>(st, a);
}

template <int KBP>
hipError_t launch_value_inst(hipStream_t st, const ValueTableArgs &a, unsigned blocks) {
  constexpr auto kern = value_table_kernel<KBP>;
  const hipError_t err = allow_full_lds<kern>();
  if (err != hipSuccess) return err;
  const size_t lds = (size_t)64 * (tile_pitch<true>(KBP) + HP) + (size_t)kHidden * 4 + (size_t)2 * NW * 64 * 4 + (size_t)kHidden * 2 + 64 * 4;
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(NT), lds, st, a);
  return hipGetLastError();
}

hipError_t launch_market_rows(hipStream_t st, const EnvDims &d, const EnvState &s, const TableMarket &m, const TableNet &net,
                              float *P, int32_t rows, bool pairs) {
  MarketArgs a;
  a.price = m.price, a.ind = m.ind, a.W = static_cast<const u32x4 *>(net.Wm), a.b = net.b[0], a.P = P;
  a.rows = rows, a.D = d.D, a.DK = d.D * d.K, a.nkb = table_market_blocks(d.D, d.K);
  a.s_price = d.s_price, a.s_ind = d.s_ind;
  a.tau = s.tau, a.start = s.start, a.N = d.N, a.H = d.H, a.table_rows = m.rows;
  auto launch = [&](auto p, auto mode) {
    constexpr Rows MODE = (Rows)decltype(mode)::value;
    constexpr auto kern = market_rows_kernel<decltype(p)::value, MODE>;
    const hipError_t err = allow_full_lds<kern>();
    if (err != hipSuccess) return err;
    constexpr int ROWS = MODE == FEWEST ? 32 : 64;
    const size_t lds = 2 * (size_t)ROWS * tile_pitch<true>(kChunk);
    hipLaunchKernelGGL(kern, dim3((unsigned)((rows + ROWS - 1) / ROWS), MODE == MANY ? 1 : MODE == FEW ? kTiles / 4 : kTiles), dim3(NT), lds, st, a);
    return hipGetLastError();
  };
  auto launch_mode = [&](auto mode) { return pairs ? launch(std::true_type{}, mode) : launch(std::false_type{}, mode); };
  return rows <= 512 ? launch_mode(Int<FEWEST>{}) : rows <= 63 * 64 ? launch_mode(Int<FEW>{}) : launch_mode(Int<MANY>{});
}

}  // namespace

bool table_supported(const pr_config &c) {
  return c.schedule == PR_SCHED_STEPWISE && c.mlp_dtype == PR_MLP_BF16 && c.hidden == kHidden && c.n_market == 1 && c.n_agents == 1 &&
         c.n_stocks > 32 && c.n_stocks <= 128 && c.n_ind >= 1;
}

int table_market_blocks(int D, int K) { return (((D * K + 3) & ~3) + D + 15) / 16; }
int table_portfolio_blocks(int D) { return portfolio_blocks(D); }

// Rows of P: those of every env and step of two episodes, which no call of so many steps needs more of (a longer table's are formed
// by env and step there); at least 8192 of them (17 MiB) and at most 128 MiB, or one step's.  16 envs over 100 rows: 17 MiB of
// workspace, where every handle had 128.  Calls of more steps go in pieces if their table is longer than that too.
int64_t table_rows_kept(int64_t n_envs, int64_t horizon) {
  const int64_t most = ((int64_t)128 << 20) / (kPitch * 4);
  return max(n_envs, min(most, max((int64_t)8192, 2 * n_envs * horizon)));
}
size_t table_scratch_bytes(int64_t n_envs, int64_t horizon) { return (size_t)table_rows_kept(n_envs, horizon) * kPitch * 4; }

hipError_t launch_rollout_table(hipStream_t st, const EnvDims &d, const EnvState &s, const TableMarket &m, const TableNet &actor,
                                float *P, int32_t *tau0, int32_t T, const float *noise, const pr_buffers &out, int cus) {
  const int64_t kept = table_rows_kept(d.N, d.H);
  const bool pairs = m.rows > kept || (int64_t)m.rows > (int64_t)T * d.N;
  const int32_t steps = pairs ? (int32_t)min((int64_t)T, kept / d.N) : T;
  TableArgs a;
  a.d = d, a.st = s, a.price = m.price, a.ind = m.ind, a.P = P;
  a.Wp = static_cast<const u32x4 *>(actor.Wp), a.W2 = static_cast<const u32x4 *>(actor.W[1]), a.W3 = static_cast<const u32x4 *>(actor.W[2]);
  a.b2 = actor.b[1], a.b3 = actor.b[2];
  a.nct3 = (d.D + 31) / 32;
  a.pairs = pairs;
  const int rounds = (d.N + 32 * cus - 1) / (32 * cus);
  a.per = max(1, (d.N + rounds * cus - 1) / (rounds * cus));
  const size_t N = (size_t)d.N, D = (size_t)d.D, S = (size_t)d.S;
  for (int32_t t = 0; t < T; t += steps) {
    a.T = min(steps, T - t);
    a.p_rows = pairs ? a.T * d.N : m.rows;
    if (t == 0 || pairs) {
      const hipError_t err = launch_market_rows(st, d, s, m, actor, P, a.p_rows, pairs);
      if (err != hipSuccess) return err;
    }
    a.first = t == 0;
    a.tau0 = t == 0 ? tau0 : nullptr;
    a.noise = noise + t * N * D;
    a.obs = out.obs + t * N * S;
    a.act_raw = out.act_raw + t * N * D;
    a.reward = out.reward + t * N;
    a.done = out.done + t * N;
    a.logp = out.logp ? out.logp + t * N : nullptr;
    a.mu = out.mu ? out.mu + t * N * D : nullptr;
    a.shares = out.shares ? out.shares + t * N * D : nullptr;
    const hipError_t err = with_blocks(d.D, [&](auto k) { return launch_rollout_blocks<decltype(k)::value>(st, a); });
    if (err != hipSuccess) return err;
  }
  return hipSuccess;
}

// Its two launches take 18 us over a short table's rows at the least and 26 over 3000, whatever the observations; for few of them the
// kernels for any network are faster: query_kernel (up to 8192 rows of 640 inputs), or a launch per layer (1024 rows of more).  us of the
// value head, this -> those, tables of 33 rows:
//   rows            80            600           2000           3400           5000           7500
//   161 inputs 18.1 ->  9.0  18.1 ->  9.1  18.2 ->  9.3  18.4 ->  9.6  18.4 -> 18.0  18.7 -> 18.2
//   401        20.2 -> 11.5  20.1 -> 11.5  19.8 -> 11.5  20.3 -> 11.9  20.0 -> 23.1  20.8 -> 24.7
//   1001       25.6 -> 13.5  25.8 -> 20.6  26.1 -> 57.4
// and of 400 rows 161 inputs 5000 rows 21.3 -> 18.1, 401 inputs 24.8 -> 25.7; of 3000 rows 7500 rows 26.2 -> 19.1, 27.0 -> 24.1.
// Tables of more than half the rows are worth their sums where those kernels are far slower: more than 640 inputs, calls of one step
// with values, 100 stocks x 8, 600 envs over 2000 and 16384 rows 100 -> 68.5 and 101 -> 82, 8000 over 16384 137 -> 118; 86 x 6, 600 over 16384
// 83 -> 72 (1000 envs x 100 x 8 over 3000 rows: 94.6 before there were table sums, 101 with them in the policy alone).
bool value_table_covers(int64_t rows, int S, int32_t n_envs, int32_t horizon, int32_t table_rows) {
  const int64_t few = S > 640 ? 1024 : table_rows > 256 ? 8192 : 4096;
  const int64_t most = max(rows / 2, (int64_t)(S > 640 ? 16384 : 0));
  return table_rows <= min(most, table_rows_kept(n_envs, horizon)) && rows > few;
}

hipError_t launch_value_table(hipStream_t st, const EnvDims &d, const EnvState &s, const TableMarket &m, const TableNet &critic,
                              float *P, const int32_t *tau0, int64_t rows, const float *obs, float *Y, int cus) {
  hipError_t err = launch_market_rows(st, d, s, m, critic, P, m.rows, false);
  if (err != hipSuccess) return err;
  ValueTableArgs a;
  a.d = d, a.obs = obs, a.rows = rows, a.P = P, a.p_rows = m.rows, a.tau0 = tau0, a.start = s.start;
  a.Wp = static_cast<const u32x4 *>(critic.Wp), a.W2 = static_cast<const u32x4 *>(critic.W[1]);
  a.w3 = static_cast<const __bf16 *>(critic.W[2]), a.b2 = critic.b[1], a.b3 = critic.b[2], a.Y = Y;
  const int64_t tiles = (rows + 63) / 64;
  const unsigned blocks = (unsigned)(tiles < cus ? tiles : cus);
  return with_blocks(d.D, [&](auto k) { return launch_value_inst<decltype(k)::value>(st, a, blocks); });
}

}  // namespace pod
