// One PPO minibatch of the learner (Sec. 4.2 "Learner": fetch a batch of
// transitions from the buffer, train the networks; Sec. 5.2: PPO, batch size
// 1024, learning rate 1e-3): forward of actor and critic with the activations
// kept, clipped-surrogate and value loss, backward through both 3-layer
// perceptrons, Adam.  fp32 master weights and activations.
//
// A step is six launches, each over both networks:
//   1. h1 = tanh(X W1 + b1), the minibatch rows gathered as they are read
//   2. h2 = tanh(h1 W2 + b2)
//   3. output layers, losses, dz3, and dz2 = (dz3 W3') (1 - h2^2)
//   4. dz1 = (dz2 W2') (1 - h1^2)  and  gW2 = h1' dz2, gb2
//   5. gW1 = X' dz1, gb1  and  gW3 = h2' dz3, gb3
//   6. partial sums of the split weight gradients added up (in order), Adam
// At the paper's batch of 1024 nothing is large: what a step costs is launches
// and the memory round trips inside each, so independent products share a launch
// and no launch does anything that the next could do while it reads.
//
// The forward pass keeps one fp32 accumulator per element (see forward_kernel).  The backward products run on the
// bf16 matrix instructions without giving up binary32 precision: an fp32 number is exactly the sum of three bf16
// numbers, and of the nine products the six that are not below 2^-26 of the result are summed in fp32 -- what is
// dropped is smaller than the rounding of one fp32 product (pod_split3.h).  Six bf16 instructions take 6/16 of the time
// of the fp32 instruction's same work.  2-norm errors against 64 bits, relative to the fp32 instructions' (batches from
// 256 to 32768, 64 to 512 units): gW1 0.72, gW2 0.71, gW3 0.89, gb1 0.91, the others as before.
//
// Measured (301-512-512 networks): a step at batch 1024 84 us (315 us as 38 launches); gradients at 15000 samples with
// 256 hidden units 277 us (753 us).
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "pod_internal.h"
#include "pod_split3.h"

namespace pod {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef f32x4 f32x4u __attribute__((aligned(4)));
typedef f32x2 f32x2u __attribute__((aligned(4)));

// ------------------------------------------------------------------ dense products
// C[M, N] = A' B' with k running over K.  Operand layouts by kind:
//   DZ   A'[m][k] = A[m lda + k]   B'[k][n] = B[n ldb + k]     (dz x transposed weights)
//   DW   A'[m][k] = A[k lda + m]   B'[k][n] = B[k ldb + n]     (transposed activations x dz; k is the batch)
// `gather`: rows of A (indexed by k, DW) are rows gather[.] of the buffer.
enum Kind { DZ = 1, DW = 2 };

struct Prob {
  const float *A, *B;
  const int32_t *gather;
  float *C;              // DZ: [M, N];  DW: the first split's part of gW
  const float *aux;      // DZ: C = . * (1 - aux^2)
  float *colsum;         // DW: the first split's part of gb[n] = sum_k B'[k][n]
  float *part;           // DW: later splits, [split - 1][M + 1][N], the column sums in row M
  int64_t lda;
  int32_t ldb, ldc, M, N, K;    // ldc: rows of C and aux (the later splits' parts are dense)
  int32_t kind, tiles_n, tiles, splits, k_chunk;
  int32_t first_block, blocks;  // blocks = tiles * splits rounded up to a multiple of 8
};
constexpr int kMaxProbs = 4;
constexpr int kOwnTiles = 1000;  // tiles from which every wavefront takes one of its own
struct ProbSet {
  Prob p[kMaxProbs];
  int32_t n;
};

// A wavefront computes a 64 x 64 tile of C, its operands read straight from global memory into the registers of the
// matrix operands: no LDS and no barrier in the loop.  With fewer tiles than SIMDs the eight wavefronts of a
// workgroup share one tile's k range (every operand element is still read by exactly one of them) and their
// accumulators are added up, in order, in LDS at the end; with more, each wavefront takes a tile of its own, or four of
// them share operands (wide_product).
// Operand of a 32 x 32 x 16 product: lane l holds 8 consecutive k of row (column) l % 32, k group l / 32.
//   k contiguous in memory: four requests of 16 rows x 64 bytes, whose lane quarters then exchange halves; row of block x
//   is 32 x + l % 32.  (A lane that reads its own eight k asks for two pieces of 32 rows each: 104 to 137 cycles of the
//   compute unit a request from L2, where 16 rows x 64 bytes take 33.)
//   m (n) contiguous: eight 8-byte loads, one per k, that serve both 32-row blocks: row of block x is 2 (l % 32) + x.
constexpr int kTile = 64, kPitch = kTile + 4;

// Granularity is 16 k (one matrix instruction deep).  Requests are made for ascending k: `load` reads the 16 k at the
// present position into a slot, `advance` moves on.
template <class T>
__device__ inline void pin(T &x) { asm volatile("" : "+v"(x)); }  // x is needed, and settled, here

// lo's odd lane quarters exchanged with hi's even ones
__device__ inline void swap_quarters(float lo, float hi, float &even, float &odd) {
  const auto s = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi), false, false);
  const uint32_t s0 = s[0], s1 = s[1];
  even = __builtin_bit_cast(float, s0), odd = __builtin_bit_cast(float, s1);
}

template <int SLOTS>
struct RawK {  // k-contiguous operand: [slot][group of 16 rows][4]
  const float *base;  // uniform
  uint32_t off[4];    // of row l % 16 of each group, k quarter l / 16
  f32x4 v[SLOTS][4];
  __device__ void init(const float *b, int64_t ld, int r0, int rows, const int32_t *, int k, int, int lane) {
    base = b + r0 * ld + k;
#pragma unroll
    for (int z = 0; z < 4; ++z) off[z] = (uint32_t)(min(r0 + 16 * z + (lane & 15), rows - 1) - r0) * (uint32_t)ld + 4 * (lane >> 4);
  }
  template <int SLOT>
  __device__ void load(int, int, int) {
#pragma unroll
    for (int z = 0; z < 4; ++z) v[SLOT][z] = *reinterpret_cast<const f32x4u *>(base + off[z]);
  }
  __device__ void advance(int step) { base += step; }
  __device__ void next_group(int) {}
  template <int SLOT>
  __device__ void arrived() {  // (a use of the slot: the wait for it stands here)
#pragma unroll
    for (int z = 0; z < 4; ++z) pin(v[SLOT][z]);
  }
  // the eight k of block x's row l % 32: the lane quarters exchange halves of two groups of rows
  template <int SLOT>
  __device__ void take(int x, float (&out)[8]) const {
#pragma unroll
    for (int e = 0; e < 4; ++e) swap_quarters(v[SLOT][2 * x][e], v[SLOT][2 * x + 1][e], out[e], out[4 + e]);
  }
};

template <int SLOTS, bool GATHER, int GROUP>
struct RawM {  // m- (n-) contiguous operand: [slot][8] pairs
  static constexpr int group = 16 * GROUP;  // k of a group of steps
  const float *base;  // uniform
  const int32_t *gather;
  uint32_t off;       // of this lane's column pair and k half
  int64_t ld;
  int k, kend;
  int32_t ids[2];  // GATHER: rows of the present group of steps (at most 64 k) and of the next one, a lane each
  bool second;    // the pair was moved down by one at the end of the row: its first element is the second loaded
  f32x2 v[SLOTS][8];
  __device__ int32_t rows_from(int k0, int lane) const { return gather[min(k0 + lane, kend - 1)]; }
  __device__ void init(const float *b, int64_t ld_, int c0, int cols, const int32_t *g, int k_, int kend_, int lane) {
    const int c = c0 + 2 * (lane & 31), last = cols > 1 ? cols - 2 : 0;
    second = c == cols - 1 && cols > 1;
    ld = ld_, gather = g, k = k_, kend = kend_;
    off = (uint32_t)min(c, last);
    if constexpr (GATHER) {
      base = b;
      ids[0] = rows_from(k, lane), ids[1] = rows_from(k + group, lane);
    } else {
      base = b + k * ld;
      off += (uint32_t)(8 * (lane >> 5)) * (uint32_t)ld;
    }
  }
  template <int SLOT>
  __device__ void load(int which, int step, int lane) {  // (which, step: GATHER, position of the step's rows in `ids`)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if constexpr (GATHER)
        v[SLOT][e] = *reinterpret_cast<const f32x2u *>(base + (__shfl(ids[which], 16 * step + 8 * (lane >> 5) + e) * ld + off));
      else
        v[SLOT][e] = *reinterpret_cast<const f32x2u *>(base + e * ld + off);
    }
  }
  __device__ void advance(int step) {
    if constexpr (!GATHER) k += step, base += step * ld;
  }
  __device__ void next_group(int lane) {
    if constexpr (GATHER) k += group, ids[0] = ids[1], ids[1] = rows_from(k + group, lane);
  }
  // the 16 k at the present position with rows outside [k_from, kend) as zeros (the others clamped into the range)
  template <int SLOT>
  __device__ void load_trimmed(int k_from, int lane) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int kk = k + 8 * (lane >> 5) + e;
      const bool ok = kk >= k_from && kk < kend;
      const int64_t row = min(kk, kend - 1);
      const int64_t at = GATHER ? (int64_t)gather[row] * ld + off : (row - k) * ld + (int64_t)(off - (uint32_t)(8 * (lane >> 5)) * (uint32_t)ld);
      const f32x2 t = *reinterpret_cast<const f32x2u *>(base + at);
      v[SLOT][e] = f32x2{ok ? t[0] : 0.0f, ok ? t[1] : 0.0f};
    }
  }
  template <int SLOT>
  __device__ void arrived() {
#pragma unroll
    for (int e = 0; e < 8; ++e) pin(v[SLOT][e]);
  }
  template <int SLOT>
  __device__ float get(int x, int e) const { return x == 0 && !second ? v[SLOT][e][0] : v[SLOT][e][1]; }
  template <int SLOT>
  __device__ void take(int x, float (&out)[8]) const {
#pragma unroll
    for (int e = 0; e < 8; ++e) out[e] = get<SLOT>(x, e);
  }
};

// kw = 1 (weight gradients): the whole range, two or three steps requested ahead; the two wavefronts of a SIMD overlap each
// other's matrix instructions (24 of 32 cycles for 16 k) and splits (about 290 vector instructions).
// kw = 8: a share of at most SLOTS 16-deep steps at a time, all requested at once; what counts is one memory round trip.
// SLOTS = 4 asks for four in any case (a branch around a request makes the compiler wait for all of them before the
// first product: 28.8 us for 26.7 at 1024 samples x 512 units).  A request is 32 scattered lines, though, and where no
// share is deeper than two steps the ones nobody uses cost more than that: SLOTS = 2 asks only for what is there (300
// samples x 256 units, launches 4 and 5 together 16.5 us for 20.2; 4096 x 128, 23.3 for 28.4).
template <int KW, int SLOTS_, Kind KIND, bool SUMS, bool GATHER>
__device__ inline void product(const Prob &g, int m0, int n0, int kbeg, int kend, int split, float *lds) {
  const int tid = threadIdx.x, lane = tid & 63, w = KW == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr bool A_K = KIND == DZ, B_K = A_K;
  constexpr int SLOTS = KW == 1 ? (GATHER ? 2 : 3) : SLOTS_;
  f32x16 acc[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[x][y][i] = 0.0f;
  float cs[2] = {0.0f, 0.0f};
  // wavefront w: the w-th share of the full 16-deep steps; what is left over goes to the last wavefront
  const int steps = (kend - kbeg) / 16, rest = (kend - kbeg) & 15, per = (steps + KW - 1) / KW;
  const int s0 = min(w * per, steps), s1 = min(s0 + per, steps);
  constexpr int GROUP = KW == 1 ? 4 : SLOTS;  // steps whose rows' indices are read at once (GATHER)
  std::conditional_t<A_K, RawK<SLOTS>, RawM<SLOTS, GATHER, GROUP>> ra;
  std::conditional_t<B_K, RawK<SLOTS>, RawM<SLOTS, false, GROUP>> rb;
  bf16x8 a[2][3], b[2][3];  // [block][part]
  // The matrix instructions drop what does not fit into an accumulator towards minus infinity, about 2^-28 of the terms'
  // magnitude: nothing in a product, but gb1 adds dz1 up over the batch, and there it adds up too (2-norm error of gb1 at
  // 16384 samples x 64 units 1.3e-6; 3.6e-7 with fp32 instructions, which round to nearest, and as it is now).  So DZ forms
  // the odd rows, every second sample, negated.
  const uint32_t flip = (uint32_t)lane << 31;
  auto split_slot = [&](auto slot) {
    constexpr int SL = decltype(slot)::value;
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      float va[8], vb[8];
      ra.template take<SL>(x, va);
      rb.template take<SL>(x, vb);
      if constexpr (KIND == DZ) {
#pragma unroll
        for (int e = 0; e < 8; ++e) va[e] = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, va[e]) ^ flip);
      }
      split3(va, a[x]);
      split3(vb, b[x]);
    }
  };
  auto add_sums = [&](auto slot) {
    constexpr int SL = decltype(slot)::value;
    if constexpr (SUMS) {
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int e = 0; e < 8; ++e) cs[x] += rb.template get<SL>(x, e);
    }
  };
  auto multiply = [&] {
#pragma unroll
    for (int q = 0; q < 6; ++q) {
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
          acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[x][kSplitA[q]], b[y][kSplitB[q]], acc[x][y], 0, 0, 0);
    }
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, SLOTS >= 3 ? 2 : 0>;
  using I3 = std::integral_constant<int, SLOTS == 4 ? 3 : 0>;
  // (requests past the wavefront's last step repeat it)
  auto load = [&](auto slot, bool more, int which, int step) {
    ra.template load<decltype(slot)::value>(which, step, lane);
    rb.template load<decltype(slot)::value>(which, step, lane);
    ra.advance(more ? 16 : 0);
    rb.advance(more ? 16 : 0);
  };
  if (s0 < s1) {
    const int k0 = kbeg + 16 * s0;
    ra.init(g.A, g.lda, m0, g.M, g.gather, k0, kend, lane);
    rb.init(g.B, g.ldb, n0, g.N, nullptr, k0, kend, lane);
    if constexpr (KW == 1) {
      // Rounds, and what is left of one behind the loop: with the way out inside it the compiler waits for everything
      // requested at its head.
      auto step = [&](auto cur, int s, bool request, int which, int at) {
        split_slot(cur);
        if (SUMS) add_sums(cur);
        if (request) load(cur, s + SLOTS + 1 < s1, which, at);
        multiply();
        __builtin_amdgcn_sched_barrier(0);
      };
      int s = s0;
      load(I0{}, s0 + 1 < s1, 0, 0);
      load(I1{}, s0 + 2 < s1, 0, 1);
      if constexpr (GATHER) {
        for (; s + 4 <= s1; s += 4) {
          step(I0{}, s, true, 0, 2);
          step(I1{}, s + 1, true, 0, 3);
          step(I0{}, s + 2, true, 1, 0);
          step(I1{}, s + 3, true, 1, 1);
          ra.next_group(lane);
        }
        if (s < s1) step(I0{}, s, true, 0, 2);
        if (s + 1 < s1) step(I1{}, s, false, 0, 0);
        if (s + 2 < s1) step(I0{}, s, false, 0, 0);
      } else {
        load(I2{}, s0 + 3 < s1, 0, 0);
        for (; s + 3 <= s1; s += 3) {
          step(I0{}, s, true, 0, 0);
          step(I1{}, s + 1, true, 0, 0);
          step(I2{}, s + 2, true, 0, 0);
        }
        if (s < s1) step(I0{}, s, false, 0, 0);
        if (s + 1 < s1) step(I1{}, s, false, 0, 0);
      }
    } else {
      for (int s = s0; s < s1; s += SLOTS) {
        load(I0{}, s + 1 < s1, 0, 0);
        if (SLOTS == 4 || s + 1 < s1) load(I1{}, s + 2 < s1, 0, 1);
        if constexpr (SLOTS == 4) {
          load(I2{}, s + 3 < s1, 0, 2);
          load(I3{}, s + 4 < s1, 0, 3);
        }
        ra.next_group(lane);
        auto take = [&](auto slot, int i) {
          if (s + i >= s1) return;
          split_slot(slot);
          if (SUMS) add_sums(slot);
          multiply();
        };
        take(I0{}, 0);
        take(I1{}, 1);
        if constexpr (SLOTS == 4) {
          take(I2{}, 2);
          take(I3{}, 3);
        }
      }
    }
  }
  if (rest && w == KW - 1) {
    // (DW only: the k of DZ is the hidden width.)  The last 16 of a k range that is no multiple of 16 are the 16 that
    // end it, the ones already counted as zeros in B'; a range of fewer than 16 repeats its last row, zeros likewise.
    const int k_read = max(kbeg, kend - 16);
    ra.init(g.A, g.lda, m0, g.M, g.gather, k_read, kend, lane);
    rb.init(g.B, g.ldb, n0, g.N, nullptr, k_read, kend, lane);
    if constexpr (KIND == DW) {
      ra.template load_trimmed<0>(kbeg + 16 * steps, lane);
      rb.template load_trimmed<0>(kbeg + 16 * steps, lane);
    }
    split_slot(I0{});
    if (SUMS) add_sums(I0{});
    multiply();
  }
  float *C = g.C, *C_sum = g.colsum;
  int64_t ldc = g.ldc;
  if (split > 0) C = g.part + (int64_t)(split - 1) * (g.M + 1) * g.N, C_sum = C + (int64_t)g.M * g.N, ldc = g.N;
  if constexpr (KW == 1) {
    // (weight gradients: both operands m-contiguous)  Accumulator register i of lane l: row 8 (i / 4) + 4 (l / 32) + i % 4,
    // column l % 32; the blocks interleave, so a lane's two columns are neighbours.
    const int half = lane >> 5, N = g.N, n = n0 + 2 * (lane & 31);
    const bool full = m0 + kTile <= g.M && n0 + kTile <= N;
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int m = m0 + 2 * (8 * (i >> 2) + 4 * half + (i & 3)) + x;
        float *dst = C + m * ldc + n;
        if (full) {
          *reinterpret_cast<f32x2u *>(dst) = f32x2{acc[x][0][i], acc[x][1][i]};
        } else if (m < g.M) {
          if (n < N) dst[0] = acc[x][0][i];
          if (n + 1 < N) dst[1] = acc[x][1][i];
        }
      }
    if constexpr (SUMS) {
#pragma unroll
      for (int y = 0; y < 2; ++y) {
        const float t = cs[y] + __shfl_xor(cs[y], 32);
        const int n = n0 + 2 * (lane & 31) + y;
        if (half == 0 && n < g.N) C_sum[n] = t;
      }
    }
    return;
  }
  // LDS: [wavefront][n][m], m and n in block order.
  float *mine = lds + w * (kTile * kPitch);
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 v = {acc[x][y][4 * j], acc[x][y][4 * j + 1], acc[x][y][4 * j + 2], acc[x][y][4 * j + 3]};
        *reinterpret_cast<f32x4 *>(mine + (32 * y + (lane & 31)) * kPitch + 32 * x + 8 * j + 4 * (lane >> 5)) = v;
      }
  float *lds_cs = lds + KW * (kTile * kPitch);  // [wavefront][k half][64]
  if (SUMS) {
#pragma unroll
    for (int x = 0; x < 2; ++x) lds_cs[(w * 2 + (lane >> 5)) * kTile + 32 * x + (lane & 31)] = cs[x];
  }
  // a wavefront finishes ROWS rows of the tile, lanes along n
  constexpr int ROWS = kTile / KW;
  const int n = n0 + (B_K ? lane : 2 * (lane & 31) + (lane >> 5)), nc = min(n, g.N - 1);
  auto row_of = [&](int i) {
    const int slot = ROWS * w + i;
    return m0 + (A_K ? slot : 2 * (slot & 31) + (slot >> 5));
  };
  float extra[ROWS];  // what the epilogue needs from memory, requested before the barrier
  if (A_K) {
#pragma unroll
    for (int i = 0; i < ROWS; ++i) extra[i] = g.aux[min(row_of(i), g.M - 1) * ldc + nc];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < ROWS / 4; ++q) {
    const float *src = lds + lane * kPitch + ROWS * w + 4 * q;
    f32x4 v = *reinterpret_cast<const f32x4 *>(src);
#pragma unroll
    for (int z = 1; z < KW; ++z) v += *reinterpret_cast<const f32x4 *>(src + z * (kTile * kPitch));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = row_of(4 * q + i);
      float c = KIND == DZ && (i & 1) ? -v[i] : v[i];
      if (A_K) c *= 1.0f - extra[4 * q + i] * extra[4 * q + i];
      if (n < g.N && m < g.M) C[m * ldc + n] = c;
    }
  }
  if (SUMS && w == 0 && n < g.N) {
    float t = 0.0f;
#pragma unroll
    for (int z = 0; z < 2 * KW; ++z) t += lds_cs[z * kTile + lane];
    C_sum[n] = t;
  }
}

constexpr size_t products_lds(int kw) { return kw == 1 ? 0 : (size_t)kw * (kTile * kPitch + 2 * kTile) * 4; }

// KW = 8: one tile per workgroup of eight wavefronts; KW = 1 (weight gradients): four wavefronts, a tile each (neighbours
// in n: they read the same rows of A)
template <int KW, int SLOTS>
__global__ __launch_bounds__(KW == 1 ? 256 : 512, 2) void products_kernel(ProbSet set) {
  extern __shared__ __align__(16) float lds[];
  int i = 0;
  while (i + 1 < set.n && (int)blockIdx.x >= set.p[i + 1].first_block) ++i;
  const Prob &g = set.p[i];
  // neighbouring tiles (which share rows of A) on one XCD: blocks are dealt out to the 8 XCDs in turn
  const int local = (int)blockIdx.x - g.first_block, per = g.blocks >> 3;
  int t = (local & 7) * per + (local >> 3);
  if (KW == 1) t = 4 * t + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  if (t >= g.tiles * g.splits) return;
  const int split = t / g.tiles, tile = t - split * g.tiles;
  const int tm = tile / g.tiles_n, tn = tile - tm * g.tiles_n;
  const int kbeg = split * g.k_chunk, kend = min(g.K, kbeg + g.k_chunk);
  const int m0 = tm * kTile, n0 = tn * kTile;
  if (KW == 8 && g.kind == DZ) {
    product<8, KW == 8 ? SLOTS : 2, DZ, false, false>(g, m0, n0, kbeg, kend, 0, lds);
  } else if (tm == 0) {
    if (g.gather) product<KW, SLOTS, DW, true, true>(g, m0, n0, kbeg, kend, split, lds);
    else product<KW, SLOTS, DW, true, false>(g, m0, n0, kbeg, kend, split, lds);
  } else {
    if (g.gather) product<KW, SLOTS, DW, false, true>(g, m0, n0, kbeg, kend, split, lds);
    else product<KW, SLOTS, DW, false, false>(g, m0, n0, kbeg, kend, split, lds);
  }
}

// ---- many tiles, input gradients among them: a workgroup of four wavefronts, 2 x 2 tiles of 64 x 64
// The parts of an operand are formed once for the two wavefronts that need them: wavefront w reads rows 32 w .. + 31 of
// both operands of the 128 x 128 tile, takes them apart and lays them into LDS as the matrix instructions want them: half
// the requests and half the vector instructions of a wavefront for itself.  One barrier for 16 k; the parts of the next
// 16 are formed behind the products of the present ones (six vector instructions to a matrix instruction of 32 cycles).
// Where it is long, matrix and vector work are about level and half overlapped: at 32768 samples x 512 units the matrix
// pipe is busy 53 % of the cycles, at 1.7-1.9 GHz, the vector pipe 51 %; at 15000 x 256, a tile or two to a workgroup, 41 % each
// (profiles/pmc_fp32_kernels.txt).  The launch at 15000 x 256 takes 65 us (79 with a wavefront for itself), at 32768 x 512
// 410 (484); 3000 x 512 54 (62), 33000 x 64, where half of the tile is empty, 49 (65).  The launch of weight gradients alone stays with a wavefront for
// itself: 271 or 181 rows and 30 columns leave more of 128 x 128 empty (8192 x 512 57 us for 44, 32768 x 512 196 for 185,
// 15000 x 256 60 for 64).  Operands fetched a step ahead with three buffers: 69 and 425 us in place of 65 and 410.
constexpr int kWideMix = 6;                     // vector instructions to a matrix instruction
constexpr int kWide = 128, kWideSlots = 4;      // (slots: steps of 16 k requested ahead)
constexpr int kPartBytes = kWide * 32;      // LDS: [part][k half][row][8 k] of an operand (rows side by side: no bank conflicts)
constexpr size_t kWideLds = 2 * 2 * 3 * kPartBytes;  // two buffers of both operands

// Rows (columns) 32 w .. of an operand that is contiguous along k; lane l holds k half l / 32 of row l % 32.
struct WideK {
  const float *base;  // uniform: k 0
  uint32_t off[2];
  f32x4 v[kWideSlots][2];
  __device__ void init(const float *b, int64_t ld, int r0, int rows, int, int w, int lane) {
    base = b + r0 * ld;
#pragma unroll
    for (int z = 0; z < 2; ++z)
      off[z] = (uint32_t)(min(r0 + 32 * w + 16 * z + (lane & 15), rows - 1) - r0) * (uint32_t)ld + 4 * (lane >> 4);
  }
  __device__ static int row(int place) { return place; }  // of the 32 that lane `place` (+ 32) holds
  template <int SLOT>
  __device__ void load(int k) {
#pragma unroll
    for (int z = 0; z < 2; ++z) v[SLOT][z] = *reinterpret_cast<const f32x4u *>(base + k + off[z]);
  }
  template <int SLOT>
  __device__ void take(float (&out)[8]) const {
#pragma unroll
    for (int e = 0; e < 4; ++e) swap_quarters(v[SLOT][0][e], v[SLOT][1][e], out[e], out[4 + e]);
  }
};

// The same of one that is contiguous along m (n): a lane reads pairs of neighbours of four k, and the lane quarters
// exchange: lane l holds k half l / 32 of row 2 (l % 16) + l / 16 % 2.
struct WideM {
  const float *base;
  uint32_t off;
  int64_t ld;
  int kend;
  bool second;  // the pair was moved down by one at the end of the row
  f32x2 v[kWideSlots][4];
  __device__ void init(const float *b, int64_t ld_, int c0, int cols, int kend_, int w, int lane) {
    const int c = c0 + 32 * w + 2 * (lane & 15), last = cols > 1 ? cols - 2 : 0;
    second = c == cols - 1 && cols > 1;
    base = b, ld = ld_, kend = kend_;
    off = (uint32_t)min(c, last) + (uint32_t)(4 * (lane >> 4)) * (uint32_t)ld;
  }
  __device__ static int row(int place) { return 2 * (place & 15) + (place >> 4); }
  template <int SLOT>
  __device__ void load(int k) {
    const float *at = base + k * ld;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[SLOT][i] = *reinterpret_cast<const f32x2u *>(at + i * ld + off);
  }
  // the 16 k at position k with rows outside [k_from, kend) as zeros (the others clamped into the range)
  __device__ void load_trimmed(int k, int k_from, int lane) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int kk = k + 4 * (lane >> 4) + i;
      const bool ok = kk >= k_from && kk < kend;
      const f32x2 t = *reinterpret_cast<const f32x2u *>(base + (int64_t)(min(kk, kend - 1) - 4 * (lane >> 4)) * ld + off);
      v[0][i] = f32x2{ok ? t[0] : 0.0f, ok ? t[1] : 0.0f};
    }
  }
  template <int SLOT>
  __device__ void take(float (&out)[8]) const {
#pragma unroll
    for (int i = 0; i < 4; ++i) swap_quarters(second ? v[SLOT][i][1] : v[SLOT][i][0], v[SLOT][i][1], out[i], out[4 + i]);
  }
};

template <Kind KIND, bool SUMS>
__device__ inline void wide_product(const Prob &g, int m0, int n0, int kbeg, int kend, int split, unsigned char *lds) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  constexpr bool DZ_ = KIND == DZ;
  std::conditional_t<DZ_, WideK, WideM> ra, rb;
  const int steps = max(kend - kbeg, 0) / 16, rest = max(kend - kbeg, 0) & 15;
  f32x16 acc[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[x][y][i] = 0.0f;
  float cs = 0.0f;
  const int wm = w >> 1, wn = w & 1, half = lane >> 5;
  const bool active = m0 + 64 * wm < g.M && n0 + 64 * wn < g.N;
  const uint32_t flip = (uint32_t)lane << 31;  // odd rows of DZ negated: see product
  const int place = lane & 31, half_at = half * (16 * kWide);
  unsigned char *const put_a = lds + half_at + (32 * w + place) * 16, *const put_b = put_a + 3 * kPartBytes;
  const unsigned char *const get_a = lds + half_at + (64 * wm + place) * 16;
  const unsigned char *const get_b = lds + 3 * kPartBytes + half_at + (64 * wn + place) * 16;
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  auto request = [&](auto slot, int step) {  // (past the last step: the last once more)
    const int k = kbeg + 16 * min(step, steps - 1);
    ra.template load<decltype(slot)::value>(k);
    rb.template load<decltype(slot)::value>(k);
  };
  bf16x8 pa[3], pb[3];  // parts on their way to LDS
  auto split_slot = [&](auto slot) {
    constexpr int SL = decltype(slot)::value;
    float va[8], vb[8];
    ra.template take<SL>(va);
    rb.template take<SL>(vb);
    if constexpr (DZ_) {
#pragma unroll
      for (int e = 0; e < 8; ++e) va[e] = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, va[e]) ^ flip);
    }
    if constexpr (SUMS) {
#pragma unroll
      for (int e = 0; e < 8; ++e) cs += vb[e];
    }
    split3(va, pa);
    split3(vb, pb);
  };
  auto lay = [&](int buffer) {
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      *reinterpret_cast<bf16x8 *>(put_a + buffer * (6 * kPartBytes) + j * kPartBytes) = pa[j];
      *reinterpret_cast<bf16x8 *>(put_b + buffer * (6 * kPartBytes) + j * kPartBytes) = pb[j];
    }
  };
  bf16x8 a[2][3], b[2][3];
  auto fetch = [&](int buffer) {
#pragma unroll
    for (int j = 2; j >= 0; --j)
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        a[x][j] = *reinterpret_cast<const bf16x8 *>(get_a + buffer * (6 * kPartBytes) + j * kPartBytes + x * 512);
        b[x][2 - j] = *reinterpret_cast<const bf16x8 *>(get_b + buffer * (6 * kPartBytes) + (2 - j) * kPartBytes + x * 512);
      }
  };
  auto multiply = [&] {
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
          acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[x][kSplitA[q]], b[y][kSplitB[q]], acc[x][y], 0, 0, 0);
  };
  // what this wavefront laid down is there, and everybody has read the other buffer
  auto meet = [&] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
  // ACTIVE: this wavefront's tile is not all behind the edge
  auto run = [&](auto act) {
    constexpr bool ACTIVE = decltype(act)::value;
    if (steps > 0) {
      ra.init(g.A, g.lda, m0, g.M, kend, w, lane);
      rb.init(g.B, g.ldb, n0, g.N, kend, w, lane);
      request(I0{}, 0);
      request(I1{}, 1);
      request(I2{}, 2);
      request(I3{}, 3);
      split_slot(I0{});
      lay(0);
      request(I0{}, 4);
      meet();
      // step s: products of s out of buffer s % 2, parts of s + 1 into the other, request of s + 5
      auto step = [&](auto next, int s) {
        if (ACTIVE) fetch(s & 1);
        split_slot(next);
        if (ACTIVE) multiply();
        request(next, s + 5);
        lay((s + 1) & 1);
        if (ACTIVE) {
          __builtin_amdgcn_sched_group_barrier(0x100, 12, 0);
#pragma unroll
          for (int i = 0; i < 24; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);        // a matrix instruction
            __builtin_amdgcn_sched_group_barrier(0x002, kWideMix, 0);  // vector instructions
          }
        }
        meet();
        __builtin_amdgcn_sched_barrier(0);
      };
      int s = 0;
      for (; s + 5 <= steps; s += 4) {
        step(I1{}, s);
        step(I2{}, s + 1);
        step(I3{}, s + 2);
        step(I0{}, s + 3);
      }
      auto last = [&](auto next, int i) {  // (s is a multiple of four)
        if (s + i >= steps) return;
        if (s + i + 1 < steps) split_slot(next), lay((i + 1) & 1);
        if (ACTIVE) fetch(i & 1), multiply();
        meet();
      };
      last(I1{}, 0);
      last(I2{}, 1);
      last(I3{}, 2);
      last(I0{}, 3);
    }
    if constexpr (!DZ_) {
      // (k of DZ is the hidden width.)  The last 16 of a k range that is no multiple of 16 are the 16 that end it, the ones
      // already counted as zeros on both sides; a range of fewer than 16 repeats its last, zeros likewise.
      if (rest) {
        const int k_read = max(kbeg, kend - 16);
        ra.init(g.A, g.lda, m0, g.M, kend, w, lane);
        rb.init(g.B, g.ldb, n0, g.N, kend, w, lane);
        ra.load_trimmed(k_read, kbeg + 16 * steps, lane);
        rb.load_trimmed(k_read, kbeg + 16 * steps, lane);
        split_slot(I0{});
        lay(0);
        meet();
        if (ACTIVE) fetch(0), multiply();
      }
    }
  };
  if (active) run(std::true_type{});
  else run(std::false_type{});
  float *C = g.C, *C_sum = g.colsum;
  int64_t ldc = g.ldc;
  if (split > 0) C = g.part + (int64_t)(split - 1) * (g.M + 1) * g.N, C_sum = C + (int64_t)g.M * g.N, ldc = g.N;
  if constexpr (SUMS) {
    const float t = cs + __shfl_xor(cs, 32);
    const int n = n0 + 32 * w + rb.row(place);
    if (half == 0 && n < g.N) C_sum[n] = t;
  }
  if (!active) return;
  // Accumulator register i of lane l: row in place 8 (i / 4) + 4 (l / 32) + i % 4, column in place l % 32.
  const int N = g.N, n = n0 + 64 * wn + rb.row(place);
  auto finish = [&](auto full) {
    constexpr bool FULL = decltype(full)::value;
    const int na = FULL ? n : min(n, N - 1), nb = FULL ? n + 32 : min(n + 32, N - 1);
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      auto row_of = [&](int i) { return m0 + 64 * wm + 32 * x + ra.row(8 * (i >> 2) + 4 * half + (i & 3)); };
      float h[16][2];
      if constexpr (DZ_) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float *src = g.aux + (FULL ? row_of(i) : min(row_of(i), g.M - 1)) * ldc;
          h[i][0] = src[na], h[i][1] = src[nb];
        }
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        f32x2 c = {acc[x][0][i], acc[x][1][i]};
        if constexpr (DZ_) {
          if (i & 1) c = -c;
          c = f32x2{c[0] * (1.0f - h[i][0] * h[i][0]), c[1] * (1.0f - h[i][1] * h[i][1])};
        }
        float *dst = C + row_of(i) * ldc;
        if (FULL || row_of(i) < g.M) {
          if (FULL || n < N) dst[n] = c[0];
          if (FULL || n + 32 < N) dst[n + 32] = c[1];
        }
      }
    }
  };
  if (m0 + 64 * wm + 64 <= g.M && n0 + 64 * wn + 64 <= N) finish(std::true_type{});
  else finish(std::false_type{});
}

__global__ __launch_bounds__(256, 2) void wide_products_kernel(ProbSet set) {
  __shared__ __align__(16) unsigned char lds[kWideLds];
  int i = 0;
  while (i + 1 < set.n && (int)blockIdx.x >= set.p[i + 1].first_block) ++i;
  const Prob &g = set.p[i];
  // neighbouring tiles (which share rows of A) on one XCD: blocks are dealt out to the 8 XCDs in turn
  const int local = (int)blockIdx.x - g.first_block, per = g.blocks >> 3, t = (local & 7) * per + (local >> 3);
  if (t >= g.tiles * g.splits) return;
  const int split = t / g.tiles, tile = t - split * g.tiles;
  const int tm = tile / g.tiles_n, tn = tile - tm * g.tiles_n;
  const int kbeg = split * g.k_chunk, kend = min(g.K, kbeg + g.k_chunk);
  const int m0 = tm * kWide, n0 = tn * kWide;
  if (g.kind == DZ) {
    wide_product<DZ, false>(g, m0, n0, kbeg, kend, 0, lds);
  } else if (tm == 0) {
    wide_product<DW, true>(g, m0, n0, kbeg, kend, split, lds);
  } else {
    wide_product<DW, false>(g, m0, n0, kbeg, kend, split, lds);
  }
}

// ------------------------------------------------------------------ forward
// h = tanh(A W + b) on the fp32 matrix instructions, every element one accumulator over k in ascending order (an fp32
// matrix instruction rounds after every k, so this is the fused multiply-add chain, the same bits for every tile shape
// and batch size).
// A wavefront owns 16 TX rows x 16 TY columns and reads its operands straight from global memory into registers, DEPTH - 1
// stages of 16 k ahead: no LDS and no barrier, so a SIMD's matrix unit has work whenever one of its wavefronts does.
// Bound by the fp32 matrix rate where a launch is long (32 cycles an instruction: the matrix pipe is busy 74 and 67 % of the
// cycles at 32768 samples x 512 units, 57 % at 15000 x 256, at 1.9-2.05 GHz; there the first layer takes 60 us, the tanh 5 of
// it, where slices through LDS with a barrier each took 80); otherwise by requests, of which a compute unit takes one in about 24 cycles, and by the round trips at either end.
// Three shapes (both layers together, us; slices through LDS in brackets):
//                                             2 x 4    1 x 4    1 x 1
//   15000 samples x 256 units (7504 tiles)      115      140      213    (147)
//   3000 x 512 (3008)                            80       77      120     (83)
//   1024 x 512 (1024)                                   30.3     45.2    (32.1)
//   1024 x 256 (512)                                    22.9     22.1
//   300 x 256 (152 tiles of 16 x 64)                    17.9     12.0    (12.3)
// 2 x 4 asks for 6 pieces of memory an instruction group of 32, 1 x 4 for 5 a group of 16, 1 x 1 for 5 a group of 4; with
// few tiles it is the length of one wavefront's chain that counts.
// An operand that is contiguous along k, lane (row j, q = lane / 16) with k 4 q .. 4 q + 3 of 16: swaps between the lane
// quarters give the operands of the four instructions.
__device__ inline void in_instruction_order(const f32x4 &v, float (&op)[4]) {
  uint32_t u[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float f = v[i];
    u[i] = __builtin_bit_cast(uint32_t, f);
  }
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const auto s = __builtin_amdgcn_permlane32_swap(u[p], u[2 + p], false, false);
    u[p] = s[0], u[2 + p] = s[1];
  }
#pragma unroll
  for (int p = 0; p < 4; p += 2) {
    const auto s = __builtin_amdgcn_permlane16_swap(u[p], u[p + 1], false, false);
    const uint32_t s0 = s[0], s1 = s[1];
    op[p] = __builtin_bit_cast(float, s0), op[p + 1] = __builtin_bit_cast(float, s1);
  }
}

// acc += rows of A times columns of W [K, N], k ascending.  pa: this lane's rows; nc: its (first) column.
// TY = 4: column block y is columns 4 j + y, so that a lane's weights of a row are one request; TY = 1: one block of 16.
template <int TY>
using Cols = std::conditional_t<TY == 4, f32x4, float>;
template <int TY>
using ColsU = std::conditional_t<TY == 4, f32x4u, float>;

// REST: K may be no multiple of 16.
template <int TX, int TY, int DEPTH, bool REST>
__device__ inline void stream_product(const float *const (&pa)[TX], const float *W, int N, int nc, int K, int lane,
                                      f32x4 (&acc)[TX][TY]) {
  const int q = lane >> 4;
  const uint32_t wo = (uint32_t)(q * N + nc);
  f32x4 va[DEPTH][TX], la[TX];
  Cols<TY> vb[DEPTH][4], lb[4];
  const int full = K >> 4;
  if (REST && (K & 15)) {  // what is left behind the full stages: requested first, used last
#pragma unroll
    for (int x = 0; x < TX; ++x)
#pragma unroll
      for (int i = 0; i < 4; ++i) la[x][i] = pa[x][min(16 * full + 4 * q + i, K - 1)];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      lb[i] = *reinterpret_cast<const ColsU<TY> *>(W + (int64_t)min(16 * full + 4 * i + q, K - 1) * N + nc);
    __builtin_amdgcn_sched_barrier(0);
  }
  auto request = [&](int slot, int stage) {  // (past the last one: the last once more)
    const int k = 16 * min(stage, full - 1);
#pragma unroll
    for (int x = 0; x < TX; ++x) va[slot][x] = *reinterpret_cast<const f32x4u *>(pa[x] + (k + 4 * q));
    const float *row = W + (int64_t)k * N;
#pragma unroll
    for (int i = 0; i < 4; ++i) vb[slot][i] = *reinterpret_cast<const ColsU<TY> *>(row + (int64_t)(4 * i) * N + wo);
  };
  auto multiply = [&](const f32x4 (&av)[TX], const Cols<TY> (&bv)[4]) {
    float op[TX][4];
#pragma unroll
    for (int x = 0; x < TX; ++x) in_instruction_order(av[x], op[x]);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int x = 0; x < TX; ++x)
#pragma unroll
        for (int y = 0; y < TY; ++y) {
          float b;
          if constexpr (TY == 4) b = bv[i][y];
          else b = bv[i];
          acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x4f32(op[x][i], b, acc[x][y], 0, 0, 0);
        }
  };
  if (full > 0) {
#pragma unroll
    for (int i = 0; i < DEPTH - 1; ++i) request(i, i);
    // (rounds of DEPTH stages, and what is left of one behind the loop: with the way out inside it the compiler waits for
    // everything requested at its head)
    int s = 0;
    for (; s + DEPTH <= full; s += DEPTH) {
#pragma unroll
      for (int i = 0; i < DEPTH; ++i) {
        request((i + DEPTH - 1) % DEPTH, s + i + DEPTH - 1);
        if (TX == 1) __builtin_amdgcn_sched_barrier(0);
        multiply(va[i], vb[i]);
        if (TX > 1) {
#pragma unroll
          for (int z = 0; z < TX + 4; ++z) {
            __builtin_amdgcn_sched_group_barrier(0x008, 4 * TX * TY / (TX + 4), 0);  // matrix instructions
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);                       // a request
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int i = 0; i < DEPTH - 1; ++i)
      if (s + i < full) multiply(va[i], vb[i]);
  }
  if (REST && (K & 15)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {  // zeros behind the end
#pragma unroll
      for (int x = 0; x < TX; ++x)
        if (16 * full + 4 * q + i >= K) la[x][i] = 0.0f;
      if (16 * full + 4 * i + q >= K) lb[i] = Cols<TY>{};
    }
    multiply(la, lb);
  }
}

struct FwdProb {
  const float *A, *W, *bias;
  float *C;
  int64_t lda;
};
struct FwdArgs {
  FwdProb p[2];             // actor, critic
  const int32_t *gather;    // rows of A, or null
  int32_t M, N, K, ldc, tiles_n, tiles;  // tiles: of both networks; a row of tiles is the actor's and then the critic's
  // rows copied on the side by the blocks behind the tiles: W2 of each network to rows of ldc
  const float *copy_src[2];
  float *copy_dst[2];
  int32_t first_copy, copy_rows;
};
constexpr int kFwdWaves = 4;

template <int TX, int TY, int DEPTH>
__global__ __launch_bounds__(64 * kFwdWaves, 2) void forward_kernel(FwdArgs a) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  if ((int)blockIdx.x >= a.first_copy) {
    const int row = ((int)blockIdx.x - a.first_copy) * kFwdWaves + w, net = row >= a.copy_rows, r = row - net * a.copy_rows;
    if (row < 2 * a.copy_rows)
      for (int k = lane; k < a.copy_rows; k += 64)
        a.copy_dst[net][(int64_t)r * a.ldc + k] = a.copy_src[net][(int64_t)r * a.copy_rows + k];
    return;
  }
  // neighbouring tiles (the same rows of A) in one workgroup and on one XCD
  const int per = a.first_copy >> 3, t = (((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3)) * kFwdWaves + w;
  if (t >= a.tiles) return;
  const int tm = t / (2 * a.tiles_n), tr = t - tm * 2 * a.tiles_n, net = tr >= a.tiles_n;
  const int m0 = 16 * TX * tm, n0 = 16 * TY * (tr - net * a.tiles_n);
  const FwdProb &g = a.p[net];
  const int N = a.N, K = a.K, q = lane >> 4, j = lane & 15;
  const float *pa[TX];
#pragma unroll
  for (int x = 0; x < TX; ++x) {
    int r = min(m0 + 16 * x + j, a.M - 1);
    if (a.gather) r = a.gather[r];
    pa[x] = g.A + (int64_t)r * g.lda;
  }
  const int n = n0 + TY * j, nc = min(n, N - TY);  // (N is a multiple of 32)
  const Cols<TY> bias = *reinterpret_cast<const ColsU<TY> *>(g.bias + nc);
  f32x4 acc[TX][TY];
#pragma unroll
  for (int x = 0; x < TX; ++x)
#pragma unroll
    for (int y = 0; y < TY; ++y) acc[x][y] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  stream_product<TX, TY, DEPTH, true>(pa, g.W, N, nc, K, lane, acc);
#pragma unroll
  for (int x = 0; x < TX; ++x)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = m0 + 16 * x + 4 * q + i;
      Cols<TY> c;
      if constexpr (TY == 4) {
#pragma unroll
        for (int y = 0; y < 4; ++y) c[y] = tanhf(acc[x][y][i] + bias[y]);
      } else {
        c = tanhf(acc[x][0][i] + bias);
      }
      if (m < a.M && n < N) *reinterpret_cast<Cols<TY> *>(g.C + (int64_t)m * a.ldc + n) = c;
    }
}

// ------------------------------------------------------------------ output layers and losses
struct HeadArgs {
  int32_t B, D, Hd;
  int32_t ld;                               // rows of h2 and dz2
  const float *h2[2];                       // [B, Hd]: actor, critic
  const float *W3[2], *b3[2];
  const float *act, *logp_old, *adv, *ret;  // rollout buffers, indexed through rows
  const int32_t *rows;
  float sigma, clip, value_coef;
  float *dz3[2];                            // [B, D], [B]: d L / d (last pre-activation)
  float *dz2[2];                            // [B, Hd]
  float *mu;                                // [B, D] and [B] scratch, used when a tile's means do not fit in LDS
  float *partial;                           // [blocks][4]
  int32_t net0;                             // network of blockIdx.y = 0
};
constexpr int kHeadRows = 16;
constexpr int kHeadLdsD = 1024;  // most action components whose means a workgroup keeps in LDS

// 16 samples of one network (blockIdx.y) per workgroup: output layer on the fp32 matrix cores, loss terms and the
// gradient of the last pre-activation (32 lanes per sample), then that gradient through W3' and the tanh of the second
// hidden layer.  Bound by the round trips of its stages: what the last one reads is requested at the start, and the
// output layer, one accumulator per mean over k in ascending order, is a stream of its operands without a barrier
// (1024 samples x 512 units 11.6 us, 15000 x 256 32.8; with slices of k through LDS, a barrier each, and one feature of
// four samples to a lane of the last stage, four times the requests, 19.1 and 59.4).  Three workgroups on a compute unit
// instead of two, 80 registers and three stages ahead: 12.2 and 30.6 us.
constexpr int kHeadWaves = 8, kHeadDepth = 4;
template <bool MU_LDS>
__global__ __launch_bounds__(64 * kHeadWaves, 4) void head_kernel(HeadArgs a) {
  extern __shared__ __align__(16) float lds[];
  float *s_red = lds;                               // [16][4]
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b0 = blockIdx.x * kHeadRows, net = a.net0 + blockIdx.y;
  const int B = a.B, Hd = a.Hd, D = net == 1 ? 1 : a.D;  // (D: outputs of the network)
  const int64_t ld = a.ld;
  const int row = tid >> 5, sub = tid & 31;  // the lanes of a sample in the loss
  const int b = b0 + row, bc = min(b, B - 1);
  const float inv_b = 1.0f / (float)B;
  const float *h2 = a.h2[net], *W3 = a.W3[net];
  const int64_t r = a.rows ? a.rows[bc] : bc;
  float st[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  {
    // outputs of the tile (means, or values): [16][Dp] in LDS, or the rows of the scratch
    const int Dp = MU_LDS ? D | 1 : D;
    float *mu = MU_LDS ? lds + 16 * 4 : a.mu + (int64_t)b0 * D + (net == 1 ? (int64_t)B * a.D : 0);
    const int j = lane & 15, q = lane >> 4;
    const float *h2_row = h2 + min(b0 + j, B - 1) * ld;
    // The last stage forms (dz3 W3')' tiles of 16 features x 16 samples, so that a lane has four features in a row of
    // one sample.  W3: components 4 q .. 4 q + 3 of 16 of feature row j (D < 4: from the first lane quarter).
    auto request_w3 = [&](int t, int d0) {
      const float *w3 = W3 + (int64_t)(16 * t + j) * D;
      f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
      if (D >= 4) {
        v = *reinterpret_cast<const f32x4u *>(w3 + min(d0 + 4 * q, D - 4));
      } else {
        v[0] = w3[0];
        if (D > 1) v[1] = w3[1];
        if (D > 2) v[2] = w3[2];
      }
      return v;
    };
    // the same with zeros behind the end, components that the end moved back into place
    auto in_place = [&](f32x4 v, int d0) {
      const int d = d0 + 4 * q, back = D >= 4 ? d - min(d, D - 4) : d;
      if (back & 1) v = f32x4{v[1], v[2], v[3], 0.0f};
      if (back & 2) v = f32x4{v[2], v[3], 0.0f, 0.0f};
      if (back >= 4) v = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      return v;
    };
    constexpr int PT = 2;  // tiles requested early: their first 32 components, and the activations
    f32x4 yw[PT][2], hv[PT];
    auto request = [&](int t0) {
#pragma unroll
      for (int p = 0; p < PT; ++p) {
        const int t = min(t0 + kHeadWaves * p, Hd / 16 - 1);
        yw[p][0] = request_w3(t, 0);
        if (D > 16) yw[p][1] = request_w3(t, 16);
        hv[p] = *reinterpret_cast<const f32x4 *>(h2_row + 16 * t + 4 * q);
      }
    };
    request(w);
    const float logp_old = a.logp_old[r], A = a.adv[r], ret = a.ret[r];
    const float act0 = a.act[r * a.D + min(sub, a.D - 1)];  // the first 32 components, requested early
    for (int n0 = 16 * w; n0 < D; n0 += 16 * kHeadWaves) {
      const int n = n0 + j;
      const float bias = a.b3[net][min(n, D - 1)];
      const float *const pa[1] = {h2_row};
      f32x4 acc[1][1] = {{f32x4{0.0f, 0.0f, 0.0f, 0.0f}}};
      stream_product<1, 1, kHeadDepth, false>(pa, W3, D, min(n, D - 1), Hd, lane, acc);
      if (n < D) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (MU_LDS || b0 + 4 * q + i < B)
            mu[(int64_t)(4 * q + i) * Dp + n] = net == 1 ? acc[0][0][i] + bias : tanhf(acc[0][0][i] + bias);
      }
    }
    if (!MU_LDS) __threadfence_block();
    __syncthreads();
    if (net == 1) {
      const float err = mu[(int64_t)row * Dp] - ret;
      const float dz = b < B ? a.value_coef * err * inv_b : 0.0f;
      if (sub == 0 && b < B) {
        a.dz3[1][b] = dz;
        st[1] = 0.5f * err * err * inv_b;
      }
      if (MU_LDS) {
        __syncthreads();  // (every lane of the sample has read its value)
        if (sub == 0) mu[(int64_t)row * Dp] = dz;
      }
    } else {
    float sq = 0.0f;
    if (b < B)
      for (int d = sub; d < D; d += 32) {
        const float e = (d < 32 ? act0 : a.act[r * D + d]) - mu[(int64_t)row * Dp + d];
        sq += e * e;
      }
    for (int o = 16; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 32);
    const float inv_s2 = 1.0f / (a.sigma * a.sigma);
    const float logp = -(float)D * logf(a.sigma) - 0.5f * (float)D * 1.8378770664093453f - 0.5f * sq * inv_s2;  // ln(2 pi)
    const float ratio = expf(logp - logp_old);
    const float rc = fminf(fmaxf(ratio, 1.0f - a.clip), 1.0f + a.clip);
    const float s1 = ratio * A, s2 = rc * A;
    const bool live = s1 <= s2;
    for (int d = sub; d < D; d += 32) {
      float dz = 0.0f;
      if (b < B) {
        const float m = mu[(int64_t)row * Dp + d];
        const float e = (d < 32 ? act0 : a.act[r * D + d]) - m;
        dz = (live ? -(ratio * A * e * inv_s2) * inv_b : 0.0f) * (1.0f - m * m);
        a.dz3[0][(int64_t)b * D + d] = dz;
      }
      if (MU_LDS) mu[(int64_t)row * Dp + d] = dz;
    }
    if (sub == 0 && b < B) {
      st[0] = -(live ? s1 : s2) * inv_b;
      st[2] = live ? 0.0f : inv_b;
      st[3] = ratio * inv_b;
    }
    }
    if (!MU_LDS) __threadfence_block();
    __syncthreads();
    // dz2 = (dz3 W3') (1 - h2^2): feature tiles of 16 dealt out to the wavefronts
    const float *dz = MU_LDS ? mu : a.dz3[net] + (int64_t)b0 * D;
    const float *dzrow = dz + (int64_t)(MU_LDS ? j : min(b0 + j, B - 1) - b0) * Dp;
    for (int t0 = w; t0 < Hd / 16; t0 += PT * kHeadWaves) {
      if (t0 != w) request(t0);
#pragma unroll
      for (int p = 0; p < PT; ++p) {
        const int t = t0 + kHeadWaves * p;
        if (t < Hd / 16) {
          f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
          auto add = [&](const f32x4 &v, int d0) {  // components d0 .. d0 + 15
            float op[4];
            in_instruction_order(in_place(v, d0), op);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int d = d0 + 4 * i + q;
              const float x = dzrow[min(d, D - 1)];
              acc = __builtin_amdgcn_mfma_f32_16x16x4f32(op[i], d < D ? x : 0.0f, acc, 0, 0, 0);
            }
          };
          add(yw[p][0], 0);
          if (D > 16) add(yw[p][1], 16);
          for (int d0 = 32; d0 < D; d0 += 32) {
            const f32x4 v0 = request_w3(t, d0), v1 = request_w3(t, min(d0 + 16, D));
            add(v0, d0);
            if (d0 + 16 < D) add(v1, d0 + 16);
          }
          if (b0 + j < B) {
            f32x4 c;
#pragma unroll
            for (int i = 0; i < 4; ++i) c[i] = acc[i] * (1.0f - hv[p][i] * hv[p][i]);
            *reinterpret_cast<f32x4 *>(a.dz2[net] + (int64_t)(b0 + j) * ld + 16 * t + 4 * q) = c;
          }
        }
      }
    }
  }
  if (sub == 0)
    for (int i = 0; i < 4; ++i) s_red[row * 4 + i] = st[i];
  __syncthreads();
  if (tid < 4 && (tid == 1) == (net == 1)) {
    float t = 0.0f;
    for (int g = 0; g < kHeadRows; ++g) t += s_red[g * 4 + tid];
    a.partial[(int64_t)blockIdx.x * 4 + tid] = t;
  }
}

// ------------------------------------------------------------------ sums of the split gradients, Adam
struct FinishSeg {
  float *g;                 // gradient: the first split's part, completed here
  const float *part;        // later parts, seg_stride floats apart
  float *theta, *m, *v;     // Adam (theta null: gradients only)
  int64_t n;
};
constexpr int kSegCriticB3 = 11;  // (tensors in the order W1 b1 W2 b2 W3 b3, actor first)
struct FinishArgs {
  FinishSeg seg[12];
  int64_t seg_stride[12];
  int32_t later;            // number of later parts
  float lr, b1, b2, eps, inv_c1, inv_c2;
  const float *partial;     // [blocks][4]
  int32_t blocks;
  float *stats;             // or null
  const float *dz_value;    // [batch]
  int32_t batch;
};

__device__ inline void adam_element(float g, float *theta, float *m, float *v, float lr, float b1, float b2, float eps,
                                    float inv_c1, float inv_c2) {
  const float mi = b1 * *m + (1.0f - b1) * g;
  const float vi = b2 * *v + (1.0f - b2) * g * g;
  *m = mi;
  *v = vi;
  *theta -= lr * (mi * inv_c1) / (sqrtf(vi * inv_c2) + eps);
}

// blockIdx.y = tensor; 12: the statistics (64 lanes stride the blocks, then a fixed-shape tree)
__global__ __launch_bounds__(256) void finish_kernel(FinishArgs a) {
  if (blockIdx.y == 12) {
    if (blockIdx.x != 0 || !a.stats) return;
    __shared__ float red[4][64];
    const int i = threadIdx.x >> 6, lane = threadIdx.x & 63;
    float s = 0.0f;
    for (int k = lane; k < a.blocks; k += 64) s += a.partial[(int64_t)k * 4 + i];
    red[i][lane] = s;
    __syncthreads();
    for (int o = 32; o > 0; o >>= 1) {
      if (lane < o) red[i][lane] += red[i][lane + o];
      __syncthreads();
    }
    if (lane == 0) a.stats[i] = red[i][0];
    return;
  }
  if (blockIdx.y == kSegCriticB3) {
    // The one gradient that is a single number: the sum of the value head's dz over the batch, where terms of either
    // sign cancel and the order of the sum shows.  Up to 64 chunks of the batch, four interleaved sums each, added up
    // chunk by chunk.
    if (blockIdx.x != 0) return;
    __shared__ float s_sum[64][4];
    const int chunks = min(64, (a.batch + 127) / 128), per = (a.batch + chunks - 1) / chunks;
    const int c = threadIdx.x >> 2, q = threadIdx.x & 3;
    float g = 0.0f;
    if (c < chunks) {
      const int b1 = min(a.batch, (c + 1) * per);
#pragma unroll 8
      for (int b = c * per + q; b < b1; b += 4) g += a.dz_value[b];
    }
    s_sum[c][q] = g;
    __syncthreads();
    if (threadIdx.x == 0) {
      g = 0.0f;
      for (int z = 0; z < chunks; ++z) {
        const float t = (s_sum[z][0] + s_sum[z][1]) + (s_sum[z][2] + s_sum[z][3]);
        g = z == 0 ? t : g + t;
      }
      const FinishSeg s = a.seg[kSegCriticB3];
      if (s.theta) adam_element(g, s.theta, s.m, s.v, a.lr, a.b1, a.b2, a.eps, a.inv_c1, a.inv_c2);
      else *s.g = g;
    }
    return;
  }
  const FinishSeg s = a.seg[blockIdx.y];
  const int64_t stride = a.seg_stride[blockIdx.y];
  if (a.later == 0 && !s.theta) return;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < s.n; i += (int64_t)gridDim.x * 256) {
    float g = s.g[i];
    for (int z = 0; z < a.later; ++z) g += s.part[z * stride + i];
    if (s.theta)
      adam_element(g, s.theta + i, s.m + i, s.v + i, a.lr, a.b1, a.b2, a.eps, a.inv_c1, a.inv_c2);
    else
      s.g[i] = g;
  }
}

__global__ __launch_bounds__(256) void adam_kernel(int64_t n, float *__restrict__ theta, const float *__restrict__ g,
                                                   float *__restrict__ m, float *__restrict__ v, float lr, float b1,
                                                   float b2, float eps, float inv_c1, float inv_c2) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) adam_element(g[i], theta + i, m + i, v + i, lr, b1, b2, eps, inv_c1, inv_c2);
}

#define LRN(x)                      \
  do {                              \
    hipError_t e_ = (x);            \
    if (e_ != hipSuccess) return e_; \
  } while (0)

size_t align256(size_t x) { return (x + 255) / 256 * 256; }

// ------------------------------------------------------------------ scratch
constexpr size_t kStaticScratchBytes = (size_t)24 << 20;

struct Plan {
  bool together;   // both networks in every launch; else one after the other, sharing the dz buffers
  bool padded;     // activation rows, and a copy of W2, end in 16 unused floats (see row_floats)
  int splits;      // k splits of the weight gradients
  size_t bytes;
};

// A tile reads 64 rows of a few cache lines each.  Rows of 512 floats are 2 KiB apart: all of a tile's lines then fall
// on a handful of L2 channels (measured: 25 us for a product that takes 13 us with rows of 544), and rows a multiple of
// 128 bytes apart on one bank of the L1 (16 rows x 64 bytes: 62 cycles a request, 33 with rows of 528).  A step at batch
// 1024 x 512 units with rows of 544 and of 528: 88.0 and 86.0 us; gradients of 3000 to 32768 samples within half a percent.
int row_floats(int Hd, bool padded) { return padded ? Hd + 16 : Hd; }
bool wants_padding(int Hd) { return Hd % 128 == 0; }

int64_t net_params(int S, int Hd, int O) { return (int64_t)(S + 1) * Hd + (int64_t)(Hd + 1) * Hd + (int64_t)(Hd + 1) * O; }

size_t plan_bytes(int B, int Hd, int D, int S, const Plan &p) {
  const size_t f = 4, ld = row_floats(Hd, p.padded);
  size_t t = (p.together ? 8 : 6) * align256((size_t)B * ld * f) + align256((size_t)B * D * f) + align256((size_t)B * f) +
             align256((size_t)((B + kHeadRows - 1) / kHeadRows) * 4 * f);
  if (p.padded) t += 2 * align256((size_t)Hd * ld * f);
  if (D > kHeadLdsD) t += align256((size_t)B * (D + 1) * f);
  const int64_t n = net_params(S, Hd, D) + net_params(S, Hd, 1);
  return t + align256((size_t)(p.splits - 1) * n * f);
}

// What the no-allocation call states that it needs: the minibatch with gathered rows, six activation-sized buffers and
// eight partial W2 gradients.
bool static_stated(int B, int Hd, int D, int S) {
  const size_t f = 4, Sp = (size_t)(S + 3) / 4 * 4;
  return align256((size_t)B * Sp * f) + 6 * align256((size_t)B * Hd * f) + 2 * align256((size_t)B * D * f) +
             2 * align256((size_t)B * f) + align256((size_t)((B + 7) / 8) * 4 * f) + align256((size_t)8 * Hd * Hd * f) <=
         kStaticScratchBytes;
}

// The weight gradients' k (the batch) is split until a workgroup walks about 512 samples, or until there are 256
// workgroups, but in the second case not beyond 32 of a launch per XCD, which would take a second round (64 units, 301
// inputs: 22 splits 59.6 us a step at batch 4096 and 100.9 at 9800, 20 splits 55.4 and 92.9).
// Gradients for which there is the no-allocation call give that call's bits, so they have a plan that fits its scratch:
// fewer splits first, then unpadded rows, then the two networks one after the other (six instead of eight activation-sized
// buffers).  That costs up to four times the time (128 units, 7800 samples: 540 us for 116), so no other call is held to it.
Plan make_plan(int B, int Hd, int D, int S, bool adam) {
  const int nh = (Hd + 63) / 64, ns = (S + 63) / 64, no = (D + 63) / 64;
  const int64_t tiles = (int64_t)nh * (ns + nh) * 2, base = (B + 511) / 512;
  int64_t want = base;
  if (tiles * want < 256) want = std::min<int64_t>((B + 127) / 128, (256 + tiles - 1) / tiles);
  auto per_xcd = [&](int64_t w) { return 2 * ((nh * ns * w + 7) / 8) + (nh * no * w + 7) / 8 + (nh * w + 7) / 8; };
  while (want > base && per_xcd(want) > 32) --want;
  want = std::max<int64_t>(1, std::min<int64_t>(want, 32));
  Plan best{true, wants_padding(Hd), (int)want, 0};
  best.bytes = plan_bytes(B, Hd, D, S, best);
  if (adam || !static_stated(B, Hd, D, S) || best.bytes <= kStaticScratchBytes) return best;
  for (int i = 0; i < 3; ++i) {
    Plan q{i < 2, i == 0 && best.padded, 1, 0};
    if (plan_bytes(B, Hd, D, S, q) > kStaticScratchBytes) continue;
    for (q.splits = (int)want; (q.bytes = plan_bytes(B, Hd, D, S, q)) > kStaticScratchBytes; --q.splits) {}
    return q;
  }
  return best;
}

// C = products of `set`: fills in the tiling and launches
hipError_t launch_products(hipStream_t st, ProbSet &set) {
  int64_t waves = 0;
  int32_t deepest = 0;
  for (int i = 0; i < set.n; ++i) {
    Prob &p = set.p[i];
    p.tiles_n = (p.N + kTile - 1) / kTile;
    const int64_t tiles = (int64_t)((p.M + kTile - 1) / kTile) * p.tiles_n;
    if (tiles * p.splits > (1 << 30)) return hipErrorInvalidValue;
    p.tiles = (int32_t)tiles;
    p.k_chunk = p.splits > 1 ? ((p.K + p.splits - 1) / p.splits + 31) / 32 * 32 : p.K;
    waves += tiles * p.splits;
    deepest = std::max(deepest, p.k_chunk);
  }
  // a wavefront per tile when that gives most SIMDs one
  const bool own = waves >= kOwnTiles, wide = own && set.p[set.n - 1].kind == DZ;
  int32_t next = 0;
  for (int i = 0; i < set.n; ++i) {
    Prob &p = set.p[i];
    if (wide) {
      p.tiles_n = (p.N + kWide - 1) / kWide;
      p.tiles = (p.M + kWide - 1) / kWide * p.tiles_n;
    }
    const int64_t wg = own && !wide ? ((int64_t)p.tiles * p.splits + 3) / 4 : (int64_t)p.tiles * p.splits;
    p.first_block = next;
    p.blocks = (int32_t)((wg + 7) / 8 * 8);
    next += p.blocks;
  }
  if (wide) {
    hipLaunchKernelGGL(wide_products_kernel, dim3((unsigned)next), dim3(256), 0, st, set);
  } else if (own) {
    hipLaunchKernelGGL((products_kernel<1, 0>), dim3((unsigned)next), dim3(256), 0, st, set);
  } else {
    const auto shared = [&](auto slots) {
      constexpr auto *kern = products_kernel<8, decltype(slots)::value>;
      const hipError_t e = allow_full_lds<kern>();
      if (e == hipSuccess) hipLaunchKernelGGL(kern, dim3((unsigned)next), dim3(512), products_lds(8), st, set);
      return e;
    };
    // (more than two steps of 16 for one of the eight wavefronts: see product)
    LRN(deepest > 2 * 8 * 16 ? shared(std::integral_constant<int, 4>{}) : shared(std::integral_constant<int, 2>{}));
  }
  return hipGetLastError();
}

}  // namespace

size_t ppo_scratch_bytes(int B, int Hd, int D, int S, bool adam) { return make_plan(B, Hd, D, S, adam).bytes; }

hipError_t launch_ppo(hipStream_t st, const pr_ppo_config &c, const float *obs, const float *act, const float *logp_old,
                      const float *adv, const float *ret, const int32_t *rows, const pr_net_params &actor,
                      const pr_net_params &critic, const pr_net_params &ga, const pr_net_params &gc,
                      const PpoAdam *adam, void *scratch, float *stats) {
  const int B = c.batch, D = c.n_stocks, Hd = c.hidden, S = 1 + 2 * D + D * c.n_ind;
  const Plan plan = make_plan(B, Hd, D, S, adam != nullptr);
  unsigned char *sp = static_cast<unsigned char *>(scratch);
  auto take = [&](size_t floats) {
    float *r = reinterpret_cast<float *>(sp);
    sp += align256(floats * 4);
    return r;
  };
  const int ld = row_floats(Hd, plan.padded);
  const size_t act_floats = (size_t)B * ld;
  float *h1[2], *h2[2], *dz2[2], *dz1[2], *dz3[2];
  for (int i = 0; i < 2; ++i) h1[i] = take(act_floats), h2[i] = take(act_floats);
  for (int i = 0; i < 2; ++i) {
    dz2[i] = i == 0 || plan.together ? take(act_floats) : dz2[0];
    dz1[i] = i == 0 || plan.together ? take(act_floats) : dz1[0];
  }
  float *w2[2] = {nullptr, nullptr};
  if (plan.padded) w2[0] = take((size_t)Hd * ld), w2[1] = take((size_t)Hd * ld);
  dz3[0] = take((size_t)B * D), dz3[1] = take(B);
  const int blocks = (B + kHeadRows - 1) / kHeadRows;
  float *partial = take((size_t)blocks * 4);
  float *mu = D > kHeadLdsD ? take((size_t)B * (D + 1)) : nullptr;
  float *part = take(0);

  const pr_net_params *net[2] = {&actor, &critic}, *grad[2] = {&ga, &gc};
  const int out[2] = {D, 1};
  // later parts of the weight gradients: per network and layer [splits - 1][M + 1][N]
  float *parts[2][3];
  const int gm[3] = {S, Hd, Hd};
  for (int i = 0; i < 2; ++i)
    for (int l = 0; l < 3; ++l) {
      parts[i][l] = part;
      part += (size_t)(plan.splits - 1) * (gm[l] + 1) * (l < 2 ? Hd : out[i]);
    }
  auto input_grad = [&](int i) {
    Prob p{};
    p.kind = DZ, p.M = B, p.N = Hd, p.K = Hd, p.A = dz2[i], p.lda = ld, p.splits = 1, p.ldc = ld;
    p.B = plan.padded ? w2[i] : net[i]->W2, p.ldb = ld;
    p.aux = h1[i], p.C = dz1[i];
    return p;
  };
  auto weight_grad = [&](int i, int layer) {
    Prob p{};
    p.kind = DW, p.M = gm[layer], p.N = layer < 2 ? Hd : out[i], p.K = B, p.splits = plan.splits, p.part = parts[i][layer];
    if (layer == 0)
      p.A = obs, p.lda = S, p.gather = rows, p.B = dz1[i], p.C = grad[i]->W1, p.colsum = grad[i]->b1;
    else if (layer == 1)
      p.A = h1[i], p.lda = ld, p.B = dz2[i], p.C = grad[i]->W2, p.colsum = grad[i]->b2;
    else
      p.A = h2[i], p.lda = ld, p.B = dz3[i], p.C = grad[i]->W3, p.colsum = grad[i]->b3;
    p.ldb = layer < 2 ? ld : p.N, p.ldc = p.N;
    return p;
  };
  for (int layer = 0; layer < 2; ++layer) {
    FwdArgs f{};
    f.gather = layer == 0 ? rows : nullptr, f.M = B, f.N = Hd, f.K = layer == 0 ? S : Hd, f.ldc = ld;
    for (int i = 0; i < 2; ++i) {
      FwdProb &p = f.p[i];
      if (layer == 0) p.A = obs, p.lda = S, p.W = net[i]->W1, p.bias = net[i]->b1, p.C = h1[i];
      else p.A = h1[i], p.lda = ld, p.W = net[i]->W2, p.bias = net[i]->b2, p.C = h2[i];
      f.copy_src[i] = net[i]->W2, f.copy_dst[i] = w2[i];
    }
    f.copy_rows = layer == 1 && plan.padded ? Hd : 0;
    const auto launch = [&](auto kern, int tx, int ty) {
      f.tiles_n = (Hd + 16 * ty - 1) / (16 * ty);
      const int64_t tiles = (int64_t)((B + 16 * tx - 1) / (16 * tx)) * 2 * f.tiles_n;
      if (tiles > (1 << 30)) return hipErrorInvalidValue;
      f.tiles = (int32_t)tiles;
      f.first_copy = (int32_t)(((tiles + kFwdWaves - 1) / kFwdWaves + 7) / 8 * 8);
      const int blocks = f.first_copy + (2 * f.copy_rows + kFwdWaves - 1) / kFwdWaves;
      hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(64 * kFwdWaves), 0, st, f);
      return hipGetLastError();
    };
    // four tiles of 16 x 64 for every SIMD, and one for most of them: see forward_kernel
    const int64_t tiles = (int64_t)((B + 15) / 16) * ((Hd + 63) / 64) * 2;
    if (tiles >= 4096) LRN(launch(forward_kernel<2, 4, 4>, 2, 4));
    else if (tiles >= 640) LRN(launch(forward_kernel<1, 4, 6>, 1, 4));
    else LRN(launch(forward_kernel<1, 1, 8>, 1, 1));
  }
  ProbSet set{};
  HeadArgs h{};
  h.B = B, h.D = D, h.Hd = Hd, h.act = act, h.logp_old = logp_old, h.adv = adv, h.ret = ret, h.rows = rows;
  h.ld = ld, h.sigma = c.sigma, h.clip = c.clip, h.value_coef = c.value_coef, h.mu = mu, h.partial = partial;
  for (int i = 0; i < 2; ++i)
    h.h2[i] = h2[i], h.W3[i] = net[i]->W3, h.b3[i] = net[i]->b3, h.dz3[i] = dz3[i], h.dz2[i] = dz2[i];
  for (int pass = 0; pass < (plan.together ? 1 : 2); ++pass) {
    h.net0 = pass;
    const dim3 grid((unsigned)blocks, plan.together ? 2 : 1);
    const size_t lds = (16 * 4 + (D <= kHeadLdsD ? 16 * (size_t)(D | 1) : 0)) * 4;
    if (D <= kHeadLdsD) {
      LRN(allow_full_lds<head_kernel<true>>());
      hipLaunchKernelGGL(head_kernel<true>, grid, dim3(64 * kHeadWaves), lds, st, h);
    } else {
      hipLaunchKernelGGL(head_kernel<false>, grid, dim3(64 * kHeadWaves), lds, st, h);
    }
    LRN(hipGetLastError());
    set.n = 0;
    // (the longer products first: behind the others they would be what a launch ends with.  Gradients at 15000 samples x 256
    // units 282 -> 275 us, 33000 x 64 207 -> 201.5; 32768 x 512, many rounds of workgroups, 1254 -> 1268; others level)
    for (int i = pass; i < (plan.together ? 2 : pass + 1); ++i) set.p[set.n++] = weight_grad(i, 1);
    for (int i = pass; i < (plan.together ? 2 : pass + 1); ++i) set.p[set.n++] = input_grad(i);
    LRN(launch_products(st, set));
    set.n = 0;
    for (int i = pass; i < (plan.together ? 2 : pass + 1); ++i) set.p[set.n++] = weight_grad(i, 0), set.p[set.n++] = weight_grad(i, 2);
    LRN(launch_products(st, set));
  }
  FinishArgs f{};
  f.later = plan.splits - 1, f.partial = partial, f.blocks = blocks, f.stats = stats, f.dz_value = dz3[1], f.batch = B;
  int64_t nmax = 1;
  for (int i = 0; i < 2; ++i)
    for (int t = 0; t < 6; ++t) {
      const int l = t / 2, N = l < 2 ? Hd : out[i];
      FinishSeg &s = f.seg[6 * i + t];
      s.g = (&grad[i]->W1)[t];
      s.n = t % 2 == 0 ? (int64_t)gm[l] * N : N;
      s.part = parts[i][l] + (t % 2 == 0 ? 0 : (int64_t)gm[l] * N);
      f.seg_stride[6 * i + t] = (int64_t)(gm[l] + 1) * N;
      if (adam) s.theta = (&net[i]->W1)[t], s.m = (&adam->m[i]->W1)[t], s.v = (&adam->v[i]->W1)[t];
      nmax = std::max(nmax, s.n);
    }
  if (adam) {
    const double c1 = 1.0 - pow((double)c.beta1, (double)c.adam_step), c2 = 1.0 - pow((double)c.beta2, (double)c.adam_step);
    f.lr = c.lr, f.b1 = c.beta1, f.b2 = c.beta2, f.eps = c.adam_eps, f.inv_c1 = (float)(1.0 / c1), f.inv_c2 = (float)(1.0 / c2);
  }
  const int64_t bx = plan.splits == 1 && !adam ? 1 : std::min<int64_t>((nmax + 255) / 256, 1024);
  hipLaunchKernelGGL(finish_kernel, dim3((unsigned)bx, 13), dim3(256), 0, st, f);
  return hipGetLastError();
}

// ---- the same minibatch for callers that cannot allocate or own a workspace: scratch in a fixed device array
// (one copy per GPU the library runs on, held until the process ends).  In host code the array's name is only a
// stand-in for the symbol: its device address is looked up once per device and that pointer is what kernels get.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::atomic<void *> g_scratch_ptr[kMaxDevices];
}  // namespace

size_t ppo_static_scratch_bytes() { return kStaticScratchBytes; }

// make_plan needs less than stated for some shapes that are larger; where a caller is told to bring a workspace does not
// move with the plan.
bool ppo_static_covers(int B, int Hd, int D, int S) {
  return static_stated(B, Hd, D, S) && ppo_scratch_bytes(B, Hd, D, S, false) <= kStaticScratchBytes;
}

hipError_t launch_ppo_grads_static(hipStream_t st, const pr_ppo_config &c, const float *obs, const float *act,
                                   const float *logp_old, const float *adv, const float *ret, const int32_t *rows,
                                   const pr_net_params &actor, const pr_net_params &critic, const pr_net_params &ga,
                                   const pr_net_params &gc, float *stats) {
  const int S = 1 + 2 * c.n_stocks + c.n_stocks * c.n_ind;
  if (!ppo_static_covers(c.batch, c.hidden, c.n_stocks, S)) return hipErrorInvalidValue;
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  void *ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (!ptr) {
    // first call on this device (with it current): every GPU holds its own copy of the array at its own address
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev].store(ptr, std::memory_order_release);
  }
  // nothing in the scratch has to start at zero: every region is written by this call before it is read
  return launch_ppo(st, c, obs, act, logp_old, adv, ret, rows, actor, critic, ga, gc, nullptr, ptr, stats);
}

hipError_t launch_adam(hipStream_t st, int64_t n, float *theta, const float *g, float *m, float *v, float lr, float b1,
                       float b2, float eps, int32_t t) {
  const double c1 = 1.0 - pow((double)b1, (double)t), c2 = 1.0 - pow((double)b2, (double)t);
  hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, theta, g, m, v, lr, b1, b2,
                     eps, (float)(1.0 / c1), (float)(1.0 / c2));
  return hipGetLastError();
}

}  // namespace pod
