// One network layer per launch for batches up to 8192 rows that are more than launch_few_rows takes (the per-step policy
// of a few thousand envs), bf16 operands: a small-batch GEMM with the bias and tanh in its epilogue.
//
// A kernel that carries a row tile through all three layers would leave most compute units idle at these sizes.  Here a
// workgroup owns 64 rows x 128 output features of one layer (128 x 128 where those are full rounds: tall_tiles), so 2048 rows x
// 1024 features are 256 workgroups; a rollout's policy and critic stand side by side in a launch where that is one round.
#include "pod_internal.h"

#include "pod_tile.h"

namespace pod {

namespace {

using tile::f32x16;
using tile::f32x4;
using tile::u32x2;
using tile::u32x4;

constexpr int kThreads = 512;
constexpr int kFeatures = 128;

struct LayerArgs {
  // the layer of one network, or of two of the same shape side by side
  const __bf16 *X[2];  // [rows][xpitch], columns up to 16 nkb readable
  void *Y[2];          // bf16 [rows][ldy] (hidden) or fp32 [rows][ldy] (output)
  const void *W[2];    // packed weights of the layer, agent-major
  const float *b[2];   // padded biases, agent-major
  int32_t xpitch;
  int32_t rows;
  int32_t ldy;
  int64_t w_stride;    // bytes between agents
  int32_t b_stride;    // floats between agents
  int32_t out_dim, nkb, nct;
  int32_t out_tanh;
  int32_t N, envs_per_agent;
  int32_t tiles_r, tiles_f;    // row tiles and 128-feature tiles (of all networks)
  int32_t own_f;               // and of one network
  int32_t patch_r, patch_f;    // tiles per XCD in either direction
  int32_t split_f;             // XCDs side by side in the feature direction
  int32_t first_move;          // blocks from here on move indicators
};

// A wavefront moves an env's row, four groups of four indicators to a lane at a time.  Bound by HBM, which the layer's own
// workgroups leave idle; in the env step the move waited with the trades.  128 steps of 5000 envs x 100 stocks x 8 8.4 ->
// 8.0 ms, 256 of 2048 x 500 x 4 21.5 -> 21.0.
__device__ inline void move_indicators(const IndicatorMove &m, int n, int lane) {
  const int DK = m.d.D * m.d.K, NG = DK / 4;
  if (n >= m.d.N) return;
  const float *src = m.ind + (size_t)rows_of(m.d, m.s.tau[n], m.s.start[n], n).row_obs * DK;
  float *o = m.obs_next + (size_t)n * m.d.S + 1 + 2 * m.d.D;
  __bf16 *sp = reinterpret_cast<__bf16 *>(m.shadow.p) + (size_t)n * m.shadow.pitch;
  typedef f32x4 f32x4u __attribute__((aligned(4)));
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  for (int g0 = lane; g0 < NG; g0 += 4 * 64) {
    f32x4 v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = *reinterpret_cast<const f32x4u *>(src + 4 * min(g0 + 64 * i, NG - 1));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int g = g0 + 64 * i;
      if (g < NG) {
        const f32x4 y = v[i] * m.d.s_ind;
        __builtin_nontemporal_store(y, reinterpret_cast<f32x4u *>(o + 4 * g));
        *reinterpret_cast<bf16x4 *>(sp + 4 * g) = bf16x4{(__bf16)y[0], (__bf16)y[1], (__bf16)y[2], (__bf16)y[3]};
      }
    }
  }
  if (lane < (DK & 3)) {
    const float y = src[4 * NG + lane] * m.d.s_ind;
    o[4 * NG + lane] = y;
    sp[4 * NG + lane] = (__bf16)y;
  }
}

// The eight wavefronts are four k-groups of two; a group takes every fourth k-block, its wavefronts 64 rows x 64
// features each (2 x 2 accumulators of 32 x 32): an LDS operand feeds two and a weight block two matrix instructions, and
// every weight block is read by exactly one wavefront, straight into registers (RB = 4: 128 rows, 2 x 4 accumulators).  Per iteration of KI k-blocks the input
// rows pass through a double-buffered LDS tile (one barrier per iteration); weights and rows are requested a whole
// iteration before they are used, in two register sets, so the loads of the loop body are in flight behind its matrix
// instructions.  At the end the groups' partial sums are added through LDS, four accumulators at a time in pieces of 16 bytes,
// each group finishing one (numbers of 4 bytes, two at a time: 0.3 us more).
// What bounds it, 2048 rows of 3001 inputs x 1024 features, 20.8 us: per 16 k-blocks 96 KB at the 48 bytes a cycle that a
// compute unit gets (0.97 us; 64 at best) and the matrix instructions (0.5) half beside them; about 6 us before the first
// product and after the last.  Not where the bytes come from: with all requests to the same 100 KB 21.2 us, with
// rows requested an iteration earlier still 21.5.  Rows and weights straight from memory, without LDS and barriers, are bound by their
// bytes alone (15 us of a loop), but eight partial sums cost 4 us and it came out level; so did 128 rows a tile with 512
// registers a wavefront, for two networks together.
// KI = 16: 128 registers of weights and rows in flight, one workgroup per compute unit; KI = 8: half of that and two
// workgroups per compute unit, for launches with more workgroups than compute units.
// PAIR: of two networks (the choice at run time costs launches of one 0.2 us of 15 to 23).
template <int KI, int RB, bool HIDDEN, bool PAIR>
__global__ __launch_bounds__(kThreads, KI == 8 && RB == 2 ? 4 : 2) void layer_kernel(LayerArgs a, IndicatorMove move) {
  extern __shared__ __align__(16) unsigned char lds[];
  constexpr int kRows = 32 * RB;
  constexpr int LB = KI / 4;               // k-blocks per group and iteration
  constexpr int NP = KI * RB / 8;          // 16-byte pieces of the input rows per thread and iteration
  constexpr int PITCH = KI * 32 + 16;      // bytes per row of a staged chunk
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), grp = wave >> 1, half = wave & 1;

  if ((int)blockIdx.x >= a.first_move) {
    move_indicators(move, ((int)blockIdx.x - a.first_move) * (kThreads / 64) + wave, lane);
    return;
  }
  // neighbouring tiles on one XCD (block b runs on XCD b % 8): a patch of patch_r x patch_f tiles shares its L2
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int sr = slot / a.patch_f, sf = slot - sr * a.patch_f;
  const int tr = (xcd / a.split_f) * a.patch_r + sr, tile_f = (xcd % a.split_f) * a.patch_f + sf;
  if (sr >= a.patch_r || tr >= a.tiles_r || tile_f >= a.tiles_f) return;
  // (both networks' pointers arrive with the other arguments: picked by an index they would be a round trip of their own)
  const bool second = PAIR && tile_f >= a.own_f;
  const int tf = second ? tile_f - a.own_f : tile_f;
  auto own = [&](auto &two) { return second ? two[1] : two[0]; };
  const int row0 = tr * kRows;
  const int agent = (row0 % a.N) / a.envs_per_agent;
  const u32x4 *W = reinterpret_cast<const u32x4 *>(static_cast<const unsigned char *>(own(a.W)) + (size_t)agent * a.w_stride);
  const float *bias = own(a.b) + (size_t)agent * a.b_stride;
  const int nkb = a.nkb, nct = a.nct;
  const int nit = (nkb + KI - 1) / KI;

  const __bf16 *X = own(a.X);
  // input rows: piece p of the tile is 16 bytes of row p / (2 KI)
  const __bf16 *xp[NP];
  int xcol[NP], xdst[NP];
  const int last_col = nkb * 16 - 8;
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const int p = tid + kThreads * i, r = p / (2 * KI), c = p % (2 * KI);
    xp[i] = X + (size_t)min(row0 + r, a.rows - 1) * a.xpitch;
    xcol[i] = 8 * c;
    xdst[i] = r * PITCH + 16 * c;
  }
  u32x4 x[NP];
  auto load_x = [&](int it) {
#pragma unroll
    for (int i = 0; i < NP; ++i)
      x[i] = *reinterpret_cast<const u32x4 *>(xp[i] + min(xcol[i] + it * KI * 16, last_col));
  };
  auto put_x = [&](int buf) {
#pragma unroll
    for (int i = 0; i < NP; ++i) *reinterpret_cast<u32x4 *>(lds + buf * (kRows * PITCH) + xdst[i]) = x[i];
  };
  // weights: blocks KI it + 4 j + grp, feature tiles 4 tf + 2 half + {0, 1}
  const u32x4 *wp[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) wp[c] = W + (size_t)min(tf * 4 + half * 2 + c, nct - 1) * 64 + lane;
  u32x4 wa[LB][2], wb[LB][2];
  auto load_w = [&](u32x4(&w)[LB][2], int it, int j) {
    const size_t o = (size_t)min(it * KI + 4 * j + grp, nkb - 1) * nct * 64;
    w[j][0] = wp[0][o];
    w[j][1] = wp[1][o];
  };

  f32x16 acc[2][RB];
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int t = 0; t < RB; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[c][t][i] = 0.0f;
  const unsigned char *xl = lds + (lane & 31) * PITCH + 16 * (lane >> 5) + 32 * grp;
  auto mma = [&](const u32x4(&w)[LB][2], int buf, int j) {
    u32x4 v[RB];
#pragma unroll
    for (int t = 0; t < RB; ++t)
      v[t] = *reinterpret_cast<const u32x4 *>(xl + buf * (kRows * PITCH) + t * 32 * PITCH + j * 128);
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int t = 0; t < RB; ++t) tile::Op<true>::mma(w[j][c], v[t], acc[c][t]);
  };

  load_x(0);
#pragma unroll
  for (int j = 0; j < LB; ++j) load_w(wa, 0, j);
  put_x(0);
  if (nit > 1) {
    load_x(1);
#pragma unroll
    for (int j = 0; j < LB; ++j) load_w(wb, 1, j);
  }
  __syncthreads();
  // iteration it: rows of it + 1 into the other LDS buffer, rows and weights of it + 2 requested
  auto step = [&](u32x4(&w)[LB][2], int it, int buf) {
    put_x(buf ^ 1);
    load_x(it + 2);
#pragma unroll
    for (int j = 0; j < LB; ++j) {
      mma(w, buf, j);
      load_w(w, it + 2, j);
    }
    __syncthreads();
  };
  // the last two or three iterations: the k-blocks of the last one may end anywhere
  auto tail = [&](u32x4(&w)[LB][2], int it, int buf) {
    if (it + 1 < nit) put_x(buf ^ 1);
    if (it + 2 < nit) load_x(it + 2);
#pragma unroll
    for (int j = 0; j < LB; ++j) {
      if (it * KI + 4 * j + grp < nkb) mma(w, buf, j);
      if (it + 2 < nit) load_w(w, it + 2, j);
    }
    __syncthreads();
  };
  int it = 0;
  for (; it + 4 <= nit; it += 2) {
    step(wa, it, 0);
    step(wb, it + 1, 1);
  }
  tail(wa, it, 0);
  if (it + 1 < nit) tail(wb, it + 1, 1);
  if (it + 2 < nit) tail(wa, it + 2, 0);

  // -- partial sums: group g finishes accumulators g, g + 4, .. of both halves (accumulator t = feature tile t / RB, row tile
  // t % RB), PER of them a round
  constexpr int PER = KI == 8 && RB == 2 ? 2 : 4, MINE = RB / 2;
  f32x4 *red = reinterpret_cast<f32x4 *>(lds);  // [PER accumulators][3 groups][2 halves][4][64]
  f32x16 sum[MINE];
#pragma unroll
  for (int p = 0; p < 2 * RB / PER; ++p) {
    if (p) __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int t = PER * p + q, owner = t & 3;
      if (owner != grp) {
        f32x4 *d = red + ((q * 3 + (grp < owner ? grp : grp - 1)) * 2 + half) * 256 + lane;
        const f32x16 &v = acc[t / RB][t % RB];
#pragma unroll
        for (int i = 0; i < 4; ++i) d[i * 64] = f32x4{v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]};
      }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int t = PER * p + q;
      if ((t & 3) == grp) {
        f32x16 &o = sum[t >> 2];
        o = acc[t / RB][t % RB];
#pragma unroll
        for (int g = 0; g < 3; ++g) {
          const f32x4 *r = red + ((q * 3 + g) * 2 + half) * 256 + lane;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const f32x4 v = r[i * 64];
#pragma unroll
            for (int k = 0; k < 4; ++k) o[4 * i + k] += v[k];
          }
        }
      }
    }
  }
  // -- bias and tanh, then whole rows out through LDS (behind the partial sums)
  constexpr int OESZ = HIDDEN ? 2 : 4, OPITCH = kFeatures * OESZ + 16;
  unsigned char *stage = lds + PER * 24 * 1024;
#pragma unroll
  for (int m = 0; m < MINE; ++m) {
    const int t = grp + 4 * m, f0 = half * 64 + (t / RB) * 32, row = (t % RB) * 32 + (lane & 31);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int f = f0 + 8 * j + 4 * (lane >> 5);
      const f32x4 bv = *reinterpret_cast<const f32x4 *>(bias + min(tf * kFeatures + f, nct * 32 - 4));
      float y[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float z = sum[m][4 * j + i] + bv[i];
        y[i] = HIDDEN ? tile::tanh_from_scaled(z * tile::kTwoLog2e) : a.out_tanh ? tile::tanh_accurate(z) : z;
      }
      if (HIDDEN) tile::Op<true>::store4(stage + row * OPITCH + f * OESZ, y[0], y[1], y[2], y[3]);
      else *reinterpret_cast<f32x4 *>(stage + row * OPITCH + f * OESZ) = f32x4{y[0], y[1], y[2], y[3]};
    }
  }
  __syncthreads();
  const int nr = min(kRows, a.rows - row0);
  if (HIDDEN) {
    // (the hidden width is a multiple of 32: a 16-byte piece is inside or outside as a whole)
    __bf16 *Y = static_cast<__bf16 *>(own(a.Y));
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      const int p = tid + kThreads * i, r = p >> 4, c = p & 15;
      if (r < nr && tf * kFeatures + 8 * c < a.out_dim)
        *reinterpret_cast<u32x4 *>(Y + (size_t)(row0 + r) * a.ldy + tf * kFeatures + 8 * c) =
            *reinterpret_cast<const u32x4 *>(stage + r * OPITCH + 16 * c);
    }
  } else {
    float *Y = static_cast<float *>(own(a.Y));
    for (int p = tid; p < nr * kFeatures; p += kThreads) {
      const int r = p >> 7, c = p & 127;
      if (tf * kFeatures + c < a.out_dim)
        Y[(size_t)(row0 + r) * a.ldy + tf * kFeatures + c] = *reinterpret_cast<const float *>(stage + r * OPITCH + 4 * c);
    }
  }
}

// rows of X to bf16, zeros up to the end of the last k-block; one wavefront per row
__global__ __launch_bounds__(256) void rows_to_bf16_kernel(const float *__restrict__ X, int64_t ldx, int rows, int S,
                                                           int cols, __bf16 *__restrict__ out, int pitch) {
  const int lane = threadIdx.x & 63, r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= rows) return;
  const float *x = X + r * ldx;
  __bf16 *o = out + (size_t)r * pitch;
#pragma unroll 4
  for (int c = lane; c < cols; c += 64) o[c] = (__bf16)(c < S ? x[c] : 0.0f);
}

// The output layer of a value head on bf16 activations, its one feature: a wavefront per row, eight neighbouring inputs to a lane.
// Bound by the rows' bytes, which are still in the last-level cache.
constexpr int kDotRows = kThreads / 64;
__global__ __launch_bounds__(kThreads) void value_dot_kernel(const __bf16 *__restrict__ h, int pitch, int pieces, int64_t rows,
                                                            const void *W, int64_t w_stride, const float *b, int32_t b_stride, int32_t N,
                                                            int32_t envs_per_agent, float *__restrict__ Y) {
  typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
  const int lane = threadIdx.x & 63;
  const int64_t r = (int64_t)blockIdx.x * kDotRows + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  if (r >= rows) return;
  const int agent = (int)(r % N) / envs_per_agent;
  const u32x4 *w = reinterpret_cast<const u32x4 *>(static_cast<const unsigned char *>(W) + (size_t)agent * w_stride);
  const u32x4 *x = reinterpret_cast<const u32x4 *>(h + r * pitch);
  float s = 0.0f;
  for (int p = lane; p < pieces; p += 64) {
    // (packed blocks: feature 0 of inputs 16 kb + 8 g .. sits in lane 32 g)
    const bf16x8 xv = __builtin_bit_cast(bf16x8, x[p]), wv = __builtin_bit_cast(bf16x8, w[(p >> 1) * 64 + 32 * (p & 1)]);
#pragma unroll
    for (int i = 0; i < 8; ++i) s = fmaf((float)xv[i], (float)wv[i], s);
  }
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if (lane == 0) Y[r] = s + b[(size_t)agent * b_stride];
}

template <int KI, int RB, bool HIDDEN, bool PAIR = false>
hipError_t launch_layer(hipStream_t st, const LayerArgs &a, unsigned blocks, const IndicatorMove &move) {
  constexpr auto kern = layer_kernel<KI, RB, HIDDEN, PAIR>;
  constexpr int kRows = 32 * RB;
  const hipError_t e = allow_full_lds<kern>();
  if (e != hipSuccess) return e;
  const size_t chunks = 2 * (size_t)kRows * (KI * 32 + 16);
  const size_t ends = (KI == 8 && RB == 2 ? 48 : 96) * 1024 + (size_t)kRows * (kFeatures * (HIDDEN ? 2 : 4) + 16);
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(kThreads), chunks > ends ? chunks : ends, st, a, move);
  return hipGetLastError();
}

}  // namespace

// Up to 8192 rows a whole-network launch would have less than half a tile per compute unit; from 128 hidden units on a
// layer has whole feature tiles.
bool layers_supported(int64_t rows, int hidden, int bf16) { return bf16 && hidden >= 128 && rows >= 64 && rows <= 8192; }

// (the extra 64 columns keep the rows of a power-of-two width off one set of L2 channels)
int32_t layers_pitch(int cols) { return (cols + 15) / 16 * 16 + 64; }

namespace {

// An XCD's patch of tiles: the split of the eight XCDs that reads the fewest bytes (input rows and weight columns weigh the
// same per k), among those that leave the fewest tiles on the busiest XCD, up to `slots` tiles counting the same.
struct Patch {
  int split_f, r, f;
};
Patch patch_of(int tiles_r, int tiles_f, int tile_rows, int slots) {
  Patch best{};
  int best_tiles = 0, best_bytes = 0;
  for (int sf = 1; sf <= 8; sf *= 2) {
    const int pr = (tiles_r + 8 / sf - 1) / (8 / sf), pf = (tiles_f + sf - 1) / sf;
    const int tiles = pr * pf > slots ? pr * pf : slots, bytes = pr * tile_rows + pf * kFeatures;
    if (best.split_f == 0 || tiles < best_tiles || (tiles == best_tiles && bytes < best_bytes))
      best = {sf, pr, pf}, best_tiles = tiles, best_bytes = bytes;
  }
  return best;
}

// 128 rows a tile where there are more workgroups of 64 than compute units and those of 128 are one full round, or nearly: two
// thirds of the bytes for the same work, but one workgroup on a compute unit instead of two.  Rollouts, per step, tiles of 64
// rows -> this: 512 units, 7200 envs x 60 stocks (228 tiles) 47.4 -> 45.8 us, 7500 48.1 -> 46.6, 8000 49.6 -> 48.1, 7600 and 8192
// level; 1024 units, 3500 x 130 (224) 55.0 -> 52.1, 4000 57.8 -> 55.4, 4096 56.6 -> 55.7.  Two rounds are slower (8192 x 130, 1024 units
// 86.9 -> 90.4), fewer tiles too (6000 x 60, 512 units, 188 tiles 56.1 -> 57.0), and so are patches that hold a tile less on every
// XCD but read half as much again (31 x 1 tiles for 8 x 4: 7800 x 60, 512 units 47.5 -> 49.5): up to 32 tiles of an XCD are the same.
constexpr int kTallSlots = 32;  // compute units of an XCD
bool tall_tiles(int64_t rows, int64_t tiles_f, int32_t N, int32_t envs_per_agent) {
  const int64_t tall = (rows + 127) / 128 * tiles_f;
  const bool one_agent = N == envs_per_agent || envs_per_agent % 128 == 0;  // (in a tile)
  if (!one_agent || (rows + 63) / 64 * tiles_f <= 256 || tall < 224 || tall > 256) return false;
  const Patch p = patch_of((int)((rows + 127) / 128), (int)tiles_f, 128, kTallSlots);
  return p.r * p.f <= kTallSlots;
}

// Layer l of `count` networks of one shape.  `move`: indicators beside it, where there is room.
hipError_t launch_one_layer(hipStream_t st, const PackedNet *const *nets, int count, int l, int64_t rows, const ObsShadow &x, float *Y,
                            int32_t N, int32_t envs_per_agent, IndicatorMove *move) {
  const PackedNet &net = *nets[0];
  const int Hd = net.out_dim[0];
  LayerArgs a;
  for (int i = 0; i < 2; ++i) {
    const PackedNet &p = *nets[i < count ? i : 0];
    a.X[i] = static_cast<const __bf16 *>(l == 0 ? x.p : p.split_h[l - 1]);
    a.Y[i] = l == 2 ? static_cast<void *>(Y) : p.split_h[l];
    a.W[i] = p.W[l], a.b[i] = p.b[l];
  }
  a.xpitch = l == 0 ? x.pitch : layers_pitch(Hd), a.rows = (int32_t)rows;
  a.ldy = l == 2 ? net.out_dim[2] : layers_pitch(Hd);
  a.w_stride = net.w_stride[l], a.b_stride = net.b_stride[l];
  a.out_dim = net.out_dim[l], a.nkb = net.nkb[l], a.nct = net.nct[l];
  a.out_tanh = net.out_tanh;
  a.N = N, a.envs_per_agent = envs_per_agent;
  a.own_f = (net.nct[l] + 3) / 4;
  a.tiles_f = count * a.own_f;
  const bool tall = l < 2 && tall_tiles(rows, a.tiles_f, N, envs_per_agent);
  const int tile_rows = tall ? 128 : 64;
  a.tiles_r = (int32_t)((rows + tile_rows - 1) / tile_rows);
  const Patch patch = patch_of(a.tiles_r, a.tiles_f, tile_rows, tall ? kTallSlots : 1);
  a.split_f = patch.split_f, a.patch_r = patch.r, a.patch_f = patch.f;
  const unsigned blocks = 8u * (unsigned)(a.patch_r * a.patch_f);
  const bool two = blocks > 256;  // more workgroups than compute units
  a.first_move = (int32_t)blocks;
  IndicatorMove m{};
  unsigned all = blocks;
  // Indicators beside it, where half of the compute units have room for a workgroup of them (one or two are resident) and
  // the launch is long enough.  Behind full compute units they take longer than in the env step, where they wait with the
  // trades (a step of 8192 envs x 30 stocks 36.0 -> 40.7 us, of 2048 x 500 beside the second layer 64 -> 70), and longer
  // than a launch of 32 k-blocks with a workgroup on half of the compute units (2048 x 400, 512 units 51.8 -> 53.5).
  // Where they are moved: 2048 x 500 64 -> 62, 5000 x 100 53 -> 49.5, 4500 x 128 47.0 -> 45.6, 4200 x 40 36.9 -> 35.8.
  if (l > 0 && move && !move->moved && (two ? blocks <= 384 : blocks <= 128 && a.nkb >= 64)) {
    move->moved = true;
    m = *move, all += (unsigned)((m.d.N + kThreads / 64 - 1) / (kThreads / 64));
  }
  if (count == 2) {
    if (tall) return launch_layer<8, 4, true, true>(st, a, all, m);
    return two ? launch_layer<8, 2, true, true>(st, a, all, m) : launch_layer<16, 2, true, true>(st, a, all, m);
  }
  if (tall) return launch_layer<8, 4, true>(st, a, all, m);
  if (l < 2) return two ? launch_layer<8, 2, true>(st, a, all, m) : launch_layer<16, 2, true>(st, a, all, m);
  return two ? launch_layer<8, 2, false>(st, a, all, m) : launch_layer<16, 2, false>(st, a, all, m);
}

}  // namespace

bool layers_room_beside(int32_t N, int32_t envs_per_agent, int hidden) {
  const int64_t tiles_f = 2 * ((hidden + 127) / 128);
  if (((int64_t)N + 63) / 64 * tiles_f <= 256) return true;
  return hidden >= 1024 && ((int64_t)N + 127) / 128 * tiles_f <= 256 && tall_tiles(N, tiles_f, N, envs_per_agent);
}

hipError_t launch_hidden(hipStream_t st, const PackedNet &net, int64_t rows, const ObsShadow &x, int32_t N, int32_t envs_per_agent) {
  const PackedNet *nets[1] = {&net};
  for (int l = 0; l < 2; ++l) {
    const hipError_t e = launch_one_layer(st, nets, 1, l, rows, x, nullptr, N, envs_per_agent, nullptr);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_layers(hipStream_t st, const PackedNet &net, int64_t rows, const ObsShadow &x, float *Y, int32_t N,
                         int32_t envs_per_agent, IndicatorMove *move, const PackedNet *beside) {
  const PackedNet *nets[2] = {&net, beside};
  for (int l = 0; l < 3; ++l) {
    // A narrow output layer leaves few of these tiles (79 for 5000 rows x 100 stocks); workgroups of 32 features that split
    // the inputs finish sooner until their reads of the rows outweigh it.  Per step of a rollout, this kernel -> that one:
    // 8192 envs x 30 stocks, 512 units 39.9 -> 35.7 us, 1500 x 130 34.0 -> 30.7, 5000 x 100 55.4 -> 54.5, 2048 x 400 49.9 ->
    // 48.7, 600 x 500 with 1024 units 53.6 -> 50.7; 2048 x 300 with 1024 units 49.3 -> 49.5, 2048 x 500 66.0 -> 67.9.
    if (l == 2 && (rows + 63) / 64 * net.nct[2] * net.nkb[2] <= 512 * 32)
      return launch_rows_output(st, net, rows, net.split_h[1], layers_pitch(net.out_dim[0]), Y, N, envs_per_agent);
    const hipError_t e = launch_one_layer(st, nets, beside && l < 2 ? 2 : 1, l, rows, x, Y, N, envs_per_agent, move);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_value_dot(hipStream_t st, const PackedNet &net, int64_t rows, const void *h, float *Y, int32_t N, int32_t envs_per_agent) {
  hipLaunchKernelGGL(value_dot_kernel, dim3((unsigned)((rows + kDotRows - 1) / kDotRows)), dim3(kThreads), 0, st,
                     static_cast<const __bf16 *>(h), layers_pitch(net.out_dim[0]), net.out_dim[0] / 8, rows, net.W[2], net.w_stride[2],
                     net.b[2], net.b_stride[2], N, envs_per_agent, Y);
  return hipGetLastError();
}

hipError_t launch_rows_to_bf16(hipStream_t st, int64_t rows, const float *X, int64_t ldx, int S, const ObsShadow &out) {
  hipLaunchKernelGGL(rows_to_bf16_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st, X, ldx, (int)rows, S, out.cols,
                     reinterpret_cast<__bf16 *>(out.p), out.pitch);
  return hipGetLastError();
}

}  // namespace pod
