// Packed fp32 layers taken over into two fp16 parts per weight (pod_half2.h).
#include "pod_half2.h"
#include "pod_internal.h"
#include "pod_tile.h"

namespace pod {
namespace {

using tile::u32x4;

constexpr int kThreads = 1024, kWaves = kThreads / 64;
constexpr int kKept = 2;  // k-blocks of a wavefront that stay in registers

struct HalvesArgs {
  HalvesJob job[kMaxHalvesJobs];
  int32_t P, n;
};

// A workgroup per agent, layer and feature tile: the largest weight of every feature, then its weights over that, in blocks of
// the same order.  Bound by the bytes (6 in, 4 out per weight) and, for one agent, by a round trip: the hidden layers of 64
// critics of 301 inputs and 256 units 21 us, of one 5.
__global__ __launch_bounds__(kThreads) void halves_kernel(HalvesArgs a) {
  __shared__ float largest[kWaves][32];
  int id = blockIdx.x, q = 0;
  for (; q + 1 < a.n && id >= a.P * a.job[q].nct; ++q) id -= a.P * a.job[q].nct;
  const HalvesJob &jb = a.job[q];
  const int agent = id / jb.nct, ct = id - agent * jb.nct;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const bf16x8 *src = reinterpret_cast<const bf16x8 *>(static_cast<const unsigned char *>(jb.W) + (size_t)agent * jb.w_stride) + lane;
  u32x4 *dst = reinterpret_cast<u32x4 *>(static_cast<unsigned char *>(jb.H) + (size_t)agent * jb.h_stride) + lane;
  // (the three parts add up to the weight itself)
  auto fetch = [&](int kb, float (&v)[8]) {
    const bf16x8 *p = src + (size_t)(kb * jb.nct + ct) * 192;
    const bf16x8 p0 = p[0], p1 = p[64], p2 = p[128];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (float)p0[e] + ((float)p1[e] + (float)p2[e]);
  };
  float kept[kKept][8], m = 0.0f;
  auto take = [&](const float (&v)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) m = fmaxf(m, fabsf(v[e]) < __builtin_inff() ? fabsf(v[e]) : 0.0f);
  };
#pragma unroll
  for (int i = 0; i < kKept; ++i) fetch(min(w + i * kWaves, jb.nkb - 1), kept[i]);
#pragma unroll
  for (int i = 0; i < kKept; ++i) take(kept[i]);
  for (int kb = w + kKept * kWaves; kb < jb.nkb; kb += kWaves) {
    float v[8];
    fetch(kb, v);
    take(v);
  }
  m = fmaxf(m, __shfl_xor(m, 32));
  if (lane < 32) largest[w][lane] = m;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kWaves; ++i) m = fmaxf(m, largest[i][lane & 31]);
  // m in 2^e .. 2^(e + 1) goes to 2^14 .. 2^15 (numbers below 2^-86 as if they were that large)
  const int e = max((int)(__builtin_bit_cast(uint32_t, m) >> 23) - 127, -86), s = m == 0.0f ? 0 : 14 - e;
  const float scale = __builtin_bit_cast(float, (uint32_t)(127 + s) << 23);
  if (w == 0 && lane < 32)
    jb.unscale[(size_t)agent * (32 * jb.nct) + 32 * ct + lane] = __builtin_bit_cast(float, (uint32_t)(127 - s - jb.input_exp) << 23);
  auto put = [&](int kb, const float (&v)[8]) {
    f16x8 h, l;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float x = v[i] * scale;
      h[i] = half_of_nonzero(x, v[i]);
      l[i] = (_Float16)(x - (float)h[i]);
    }
    u32x4 *o = dst + (size_t)(kb * jb.nct + ct) * 128;
    o[0] = __builtin_bit_cast(u32x4, h);
    o[64] = __builtin_bit_cast(u32x4, l);
  };
#pragma unroll
  for (int i = 0; i < kKept; ++i)
    if (w + i * kWaves < jb.nkb) put(w + i * kWaves, kept[i]);
  for (int kb = w + kKept * kWaves; kb < jb.nkb; kb += kWaves) {
    float v[8];
    fetch(kb, v);
    put(kb, v);
  }
}

}  // namespace

hipError_t launch_halves(hipStream_t st, const HalvesJob *jobs, int n, int P) {
  HalvesArgs a;
  a.P = P, a.n = n;
  int64_t blocks = 0;
  for (int i = 0; i < n; ++i) a.job[i] = jobs[i], blocks += (int64_t)P * jobs[i].nct;
  if (n > kMaxHalvesJobs || blocks > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL(halves_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

}  // namespace pod
