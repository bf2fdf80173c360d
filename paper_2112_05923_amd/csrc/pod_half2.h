// fp32 numbers as sums of two fp16 numbers, for fp32 products on the fp16 matrix
// instructions: half of the matrix work and two thirds of the bytes of three bf16
// parts (pod_split3.h), for operands whose scale is known.
//
// x = h + l with h = fp16(x), l = fp16(x - h), both rounded to nearest: h takes 11
// of the 24 significant bits, the difference is exact in fp32 and has 13 with its
// sign, so the sum is x to 2^-24 |x|.  Of the four products of two split numbers
// three are formed; l l' is below 2^-24 of |x x'|, a quarter of that in the mean.  An fp32
// multiply-add leaves as much in its one rounding, and half as many products mean half
// as many roundings of the accumulator: measured against 64 bits the results are closer
// than those of three bf16 parts (figures at the kernels).
//
// fp16 ends at 65504 and has whole parts only down to 2^-14 (numbers down to 2^-24),
// so operands are scaled by powers of two first: a feature's weights by their largest
// one (to 2^14 .. 2^15), hidden activations, at most 1, by 2^14, a row of inputs by its
// largest one.  What is lost of a number far below the largest one it is added to
// is then 2^-39 of that one for weights and activations, 2^-29 for inputs.
//
// An infinity leaves h at the largest number and l infinite, a NaN one of them: l meets the
// other operand's h only, which is not zero unless the number is (half_of_nonzero).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pod {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

constexpr float kHalfMax = 65504.0f;
constexpr int kHiddenExp = 14;                // hidden activations are scaled by 2^14
constexpr float kHiddenScale = 16384.0f;

__device__ inline uint32_t half_pair(float a, float b) {
  const f16x2 v = {(_Float16)a, (_Float16)b};
  return __builtin_bit_cast(uint32_t, v);
}

// two numbers (scaled) -> two packed pairs.  SMALL: both below the largest fp16 number
template <bool SMALL>
__device__ inline void split2_pair(float a, float b, uint32_t &h, uint32_t &l) {
  auto first = [](float x) { return SMALL ? x : __builtin_amdgcn_fmed3f(x, -kHalfMax, kHalfMax); };
  h = half_pair(first(a), first(b));
  asm("" : "+v"(h));  // (settled before it is taken apart, or the compiler converts a second time)
  const f16x2 hv = __builtin_bit_cast(f16x2, h);
  l = half_pair(a - (float)hv[0], b - (float)hv[1]);
}

// h of a number that is not zero, where the scale may take it below fp16's smallest: that one
__device__ inline _Float16 half_of_nonzero(float scaled, float x) {
  const _Float16 h = (_Float16)__builtin_amdgcn_fmed3f(scaled, -kHalfMax, kHalfMax);
  return h == (_Float16)0.0f && x != 0.0f ? (_Float16)__builtin_copysignf(0x1p-24f, x) : h;
}

}  // namespace pod
