// fp32 numbers as sums of three bf16 numbers, for fp32 products on the bf16
// matrix instructions.
//
// x = x0 + x1 + x2 with x0 = bf16(x), x1 = bf16(x - x0), x2 = bf16(x - x0 - x1),
// all rounded to nearest: the differences are exact in fp32, each part takes at
// least 8 of the 24 significant bits, so the sum is x itself and |x1| <= 2^-9 |x|,
// |x2| <= 2^-18 |x|.  Of the nine products of two split numbers the six with
// i + j <= 2 are formed; the others are below 2 x 2^-27 of |x y|, less than the
// rounding of an fp32 multiply-add (2^-24), and the products that are formed are
// exact in the fp32 accumulator's input.  (Parts below the smallest normal number
// may be lost: operands smaller than about 1e-33.)
// The accumulator does not round to nearest: what does not fit is dropped towards minus infinity, 2^-28 of the terms'
// magnitude in the mean.  One result does not notice; a sum over many results does (pod_learner.hip).
//
// An infinity leaves the last part infinite and the others at 2^127, and a NaN the
// last part: the last part meets the first of the other operand only, so an infinite
// input times a finite weight is that infinity, as in fp32.  (Taken apart like the
// others it would be inf - inf = NaN in every sum it meets.  Only where an operand of
// 2^127 or more meets one above 500, beyond fp32 twice over, may the result be NaN.)
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pod {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// order of the six products: the smallest first
constexpr int kSplitA[6] = {2, 1, 0, 1, 0, 0};
constexpr int kSplitB[6] = {0, 1, 2, 0, 1, 0};

__device__ inline uint32_t bf16_pair(float a, float b) {
  const bf16x2 v = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(uint32_t, v);
}
__device__ inline float bf16_low(uint32_t p) { return __builtin_bit_cast(float, p << 16); }
__device__ inline float bf16_high(uint32_t p) { return __builtin_bit_cast(float, p & 0xffff0000u); }

// two numbers -> three packed pairs.  SMALL: both below 2^127 (tanh outputs; a NaN stays one)
template <bool SMALL = false>
__device__ inline void split3_pair(float a, float b, uint32_t &p0, uint32_t &p1, uint32_t &p2) {
  constexpr float M = 1.7014118346046923e38f;
  auto first = [](float x) { return SMALL ? x : __builtin_amdgcn_fmed3f(x, -M, M); };
  // (the packed pairs are settled before they are taken apart: left alone, the compiler converts a second time instead)
  p0 = bf16_pair(first(a), first(b));
  asm("" : "+v"(p0));
  a -= bf16_low(p0), b -= bf16_high(p0);
  p1 = bf16_pair(first(a), first(b));
  asm("" : "+v"(p1));
  a -= bf16_low(p1), b -= bf16_high(p1);
  p2 = bf16_pair(a, b);
}

// eight consecutive k of an operand row -> its three matrix operands
template <bool SMALL = false>
__device__ inline void split3(const float (&v)[8], bf16x8 (&out)[3]) {
  typedef uint32_t u32x4_ __attribute__((ext_vector_type(4)));
  u32x4_ o[3];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint32_t p0, p1, p2;
    split3_pair<SMALL>(v[2 * i], v[2 * i + 1], p0, p1, p2);
    o[0][i] = p0, o[1][i] = p1, o[2][i] = p2;
  }
#pragma unroll
  for (int j = 0; j < 3; ++j) out[j] = __builtin_bit_cast(bf16x8, o[j]);
}

}  // namespace pod
