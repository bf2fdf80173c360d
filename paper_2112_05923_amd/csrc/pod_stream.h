// fp32 networks of 256 hidden units with a wavefront per 32 rows: the weight stream of the
// value head over a long buffer.
//
// A wavefront computes all 256 features of its 32 rows, so nothing of a row ever
// leaves it: a lane of the transposed product (pod_tile.h) holds 128 of the 256
// hidden values of its row, and the k-blocks of the next layer are eight of them,
// taken apart into two fp16 numbers (pod_half2.h) right where they are consumed, under
// the matrix instructions of the block before.  No activation passes through LDS and no
// barrier stands between two layers.  What the four wavefronts of a workgroup share
// is the weights: 32 KiB chunks (48 matrix instructions per wavefront) are copied
// straight into LDS, one chunk ahead.  Per compute unit that is 22 B of weights a
// clock from L2 and 86 B a clock from LDS at the full matrix rate.
//
// Two wavefronts live on a SIMD (256 registers each), of two workgroups that keep no
// step with each other: the epilogues of one run under the matrix instructions of
// the other.  256 registers do not hold two layers of 256 features: layer 2 is
// formed in two halves of 128 features.
#pragma once

#include "pod_half2.h"
#include "pod_tile.h"

namespace pod {
namespace stream {

using namespace tile;

constexpr int kThreads = 256, kWaves = 4, kRows = 32 * kWaves;
constexpr int kBlock = 2 * 1024;       // one feature tile of a k-block: h, then l
constexpr int kChunk = 16 * kBlock;    // two k-blocks of all features or four of half of them
constexpr int kPart = kChunk / kWaves; // copied by each wavefront
constexpr int kHidden = 256;

// The eight values a lane holds of half a feature tile are a k-block of the next layer if the rows of the weight operand
// are read in the order that swaps bits 2 and 3 of the feature's index: lane (row r, half g) then holds, as accumulator
// element 8 h + e, feature 16 h + 8 g + e.
__device__ inline int operand_lane(int lane) { return (lane & ~12) | ((lane & 4) << 1) | ((lane & 8) >> 1); }

// This wavefront's part of a chunk, straight from memory into LDS (64 lanes x 16 bytes an instruction).  `src` is uniform.
// The compiler does not know of these loads: wait_chunk() waits for them.  (It would make every LDS read wait for
// the chunk that is under way.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ inline void copy_part(const unsigned char *src, uint32_t lds, uint32_t lane16) {
#pragma unroll
  for (int i = 0; i < kPart / 1024; ++i)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds + 1024 * i), "v"(lane16),
                 "s"(src + 1024 * i)
                 : "memory", "m0");
}
#pragma clang diagnostic pop

// All wavefronts are past the present chunk and the next one is complete.  LATER: how many of this wavefront's loads
// were issued behind its copies (they may stay under way).
template <int LATER>
__device__ inline void chunk_end() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(LATER) : "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// A k-block of a row, eight inputs per lane: its parts.
struct Blk2 {
  u32x4 h, l;
};

// The blocks of a chunk (the first eight of them, or all sixteen): acc(b) += block b times x(b), with work(b, i) done under the
// i-th of a block's three matrix instructions.  Four register quadruples hold the two parts of the block in use and of the one
// that follows.  Nothing moves from one instruction's work to the next: left alone, the compiler asks for every part right before
// it is used and lines the work up as chains of dependent operations.
template <class Acc, class X, class Work>
__device__ inline void chunk_products(const unsigned char *lds, bool all, Acc acc, X x, Work work) {
  u32x4 s[4];
  auto request = [&](int n) {  // part n % 2 (l first) of block n / 2
    if (n < 32) s[n & 3] = *reinterpret_cast<const u32x4 *>(lds + (n >> 1) * kBlock + (1 - (n & 1)) * 1024);
  };
#pragma unroll
  for (int n = 0; n < 2; ++n) request(n);
  auto block = [&](int b) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      if (i < 2) request(2 * b + 2 + i);
      const f16x8 w = __builtin_bit_cast(f16x8, s[(2 * b + (i > 0)) & 3]);
      f32x16 &c = acc(b);
      c = __builtin_amdgcn_mfma_f32_32x32x16_f16(w, __builtin_bit_cast(f16x8, i == 1 ? x(b).l : x(b).h), c, 0, 0, 0);
      work(b, i);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
#pragma unroll
  for (int b = 0; b < 8; ++b) block(b);
  if (all) {
#pragma unroll
    for (int b = 8; b < 16; ++b) block(b);
  }
}

// two of the eight values of an operand
template <bool SMALL>
__device__ inline void operand_pair(Blk2 &x, int pair, float a, float b) {
  uint32_t h, l;
  split2_pair<SMALL>(a, b, h, l);
  x.h[pair] = h, x.l[pair] = l;
}

}  // namespace stream
}  // namespace pod
