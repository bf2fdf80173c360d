// fp32 networks of 256 hidden units with a wavefront per 32 rows: building blocks
// shared by the value head over a long buffer and the rollout of many envs.
//
// A wavefront computes all 256 features of its 32 rows, so nothing of a row ever
// leaves it: a lane of the transposed product (pod_tile.h) holds 128 of the 256
// hidden values of its row, and the k-blocks of the next layer are eight of them,
// taken apart into three bf16 numbers right where they are consumed, under the
// matrix instructions of the block before.  No activation passes through LDS and no
// barrier stands between two layers.  What the four wavefronts of a workgroup share
// is the weights: 24 KiB chunks (48 matrix instructions per wavefront) are copied
// straight into LDS, one chunk ahead.  Per compute unit that is 16 B of weights a
// clock from L2 and 64 B a clock from LDS at the full matrix rate, where tiles of
// 64 rows shared by eight wavefronts take 32 B a clock from L2 and an epilogue in
// which the matrix cores stand still.
//
// Two wavefronts live on a SIMD (256 registers each), of two workgroups that keep no
// step with each other: the epilogues of one run under the matrix instructions of
// the other.  256 registers do not hold two layers of 256 features: layer 2 is
// formed in two halves of 128 features.
#pragma once

#include "pod_tile.h"

namespace pod {
namespace stream {

using namespace tile;

constexpr int kThreads = 256, kWaves = 4, kRows = 32 * kWaves;
constexpr int kBlock = 3 * 1024;      // one feature tile of a k-block
constexpr int kChunk = 8 * kBlock;    // eight of them
constexpr int kPart = kChunk / kWaves;  // copied by each wavefront
constexpr int kHidden = 256;
constexpr int kVectorMayPass = 0x406;  // scheduling fence for all but vector, transcendental and scalar instructions

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

// The eight blocks of a chunk: acc(b) += block b times x(b), with work(b) done under their matrix instructions.  The three
// parts of a block are used for 1, 3 and 6 of its products; four register quadruples hold what is in use and what is on
// its way, every part requested 128 or more cycles of matrix work before its first product.  Left alone, the compiler asks for
// every part right before it.
template <class Acc, class X, class Work>
__device__ inline void chunk_products(const unsigned char *lds, Acc acc, X x, Work work) {
  u32x4 s[4];
  auto request = [&](int n) {  // part n % 3 (the last one first) of block n / 3
    if (n < 24) s[n & 3] = *reinterpret_cast<const u32x4 *>(lds + (n / 3) * kBlock + (2 - n % 3) * 1024);
  };
#pragma unroll
  for (int n = 0; n < 3; ++n) request(n);
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    work(b);
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      if (i == 0) request(3 * b + 3);
      if (i == 1) request(3 * b + 4);
      if (i == 4) request(3 * b + 5);
      f32x16 &c = acc(b);
      c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, s[(3 * b + 2 - kSplitA[i]) & 3]),
                                                  __builtin_bit_cast(bf16x8, x(b).p[kSplitB[i]]), c, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(kVectorMayPass);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// two of the eight values of an operand
template <bool SMALL>
__device__ inline void operand_pair(Blk3 &x, int pair, float a, float b) {
  uint32_t p0, p1, p2;
  split3_pair<SMALL>(a, b, p0, p1, p2);
  x.p[0][pair] = p0, x.p[1][pair] = p1, x.p[2][pair] = p2;
}

}  // namespace stream
}  // namespace pod
