// A whole network in one launch for a few rows: a policy asked for actions on a handful of observations.
//
// A workgroup takes 16 rows through all three layers.  What it costs is one start of a launch, the rows' round trip, and the
// packed weights once through a compute unit's L1 -- 50 KB to 0.9 MB where a launch per layer (pod_rows.hip) pays three starts
// and three round trips instead.  A wavefront owns HD / 128 tiles of 16 features of a hidden layer with all of their inputs
// (16 x 16 x 32 instructions, the rows as their columns), its weights in a ring of requests that starts on the next
// layer before the activations of this one are formed.  Nothing is kept in memory between the layers.
#include "pod_internal.h"

#include "pod_tile.h"

namespace pod {
namespace {

using tile::f32x4;
using tile::mma16;
using tile::u32x4;
typedef f32x4 f32x4u __attribute__((aligned(4)));

constexpr int kWaves = 8, kThreads = 64 * kWaves, kRows = 16, kMaxOut = 32, kPartPitch = 36;

struct QueryArgs {
  const float *X;  // [rows][ldx]
  int64_t ldx, rows;
  PackedNet net;
  int32_t N, envs_per_agent;
  float *Y;        // [rows][out]
};

// The sums of a feature tile: input step k goes to chain k % CH.  What a sum loses it loses in its longest chain of additions:
// fp32, 301 inputs and 256 units, against 64 bits (2-norm, actor and critic, 24 networks of 1000 rows) one chain 2.2e-7 and
// 2.1e-7, two 2.0e-7 and 1.8e-7, four 1.6e-7 and 1.5e-7; a launch per layer, whose eight wavefronts split the inputs, 1.8e-7 and
// 1.7e-7.  bf16: what is lost there is far below the rounding of the operands, and two chains are as fast as one.
template <bool BF16>
struct Sums {
  static constexpr int CH = BF16 ? 2 : 4;
  f32x4 hi[CH], lo;
  __device__ inline Sums() {
#pragma unroll
    for (int k = 0; k < CH; ++k) hi[k] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    lo = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }
  __device__ inline f32x4 total() const {
    const f32x4 v = hi[0] + hi[1];
    return BF16 ? v : (v + (hi[2 % CH] + hi[3 % CH])) + lo;
  }
};

template <bool BF16>
__host__ __device__ constexpr int query_lds(int hd, int nks) {
  return kRows * (tile::tile_pitch<BF16>(2 * nks) + 2 * tile::tile_pitch<BF16>(hd / 16)) + 4 * kRows * kPartPitch * 4;
}

// PD: k-steps (of 32 inputs) of weights requested ahead
template <bool BF16, int HD, int PD>
__global__ __launch_bounds__(kThreads, 2) void query_kernel(QueryArgs a) {
  using namespace tile;
  using O = Op<BF16>;
  using Block = typename O::Block;
  constexpr int FT = HD >= 128 ? HD / 128 : 1, KS = HD / 32, NCT = HD / 32, NP = 64 * kPlanes<Block>, HP = tile_pitch<BF16>(HD / 16);
  constexpr int KP = KS >= 4 ? 4 : KS, PER = KS / KP;  // layer 3: its k-steps in KP parts
  extern __shared__ __align__(16) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t row0 = (int64_t)xcd_run(blockIdx.x, gridDim.x) * kRows;
  const Net net = net_of(a.net, (int)(row0 % a.N) / a.envs_per_agent);
  const int S = a.net.in_dim[0], nkb = net.nkb[0], nks = (nkb + 1) / 2, XP = tile_pitch<BF16>(2 * nks);
  unsigned char *ldsX = lds, *ldsH1 = ldsX + kRows * XP, *ldsH2 = ldsH1 + kRows * HP;
  float *part = reinterpret_cast<float *>(ldsH2 + kRows * HP);  // [KP][kRows][kPartPitch]
  const int q4 = lane >> 4, row = lane & 15;
  const bool active = HD >= 128 || w < HD / 16;
  const int ft0 = active ? w * FT : 0;

  // weights: packed blocks are 32 features x 16 inputs
  Block ring[PD][FT];
  auto request = [&](Block(&b)[FT], const u32x4 *W, int nblocks, int ks) {
    const int kb = min(2 * ks + (q4 >> 1), nblocks - 1);
#pragma unroll
    for (int c = 0; c < FT; ++c)
      fetch_w(b[c], W + ((size_t)kb * NCT + ((ft0 + c) >> 1)) * NP + ((ft0 + c) & 1) * 16 + row + 32 * (q4 & 1));
  };
  // -- the rows
  const int e = tid >> 5, tl = tid & 31;
  const float *x = a.X + min(row0 + e, a.rows - 1) * a.ldx;
  constexpr int GROUPS = 3;  // four columns each, requested together
  f32x4 pre[GROUPS];
  auto group = [&](int c) {
    if (c + 4 <= S) return (f32x4)*reinterpret_cast<const f32x4u *>(x + c);
    f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
    if (c < S) v[0] = x[c];
    if (c + 1 < S) v[1] = x[c + 1];
    if (c + 2 < S) v[2] = x[c + 2];
    return v;
  };
#pragma unroll
  for (int g = 0; g < GROUPS; ++g) pre[g] = group(4 * (tl + 32 * g));
#pragma unroll
  for (int s = 0; s < PD; ++s) request(ring[s], net.W[0], nkb, min(s, nks - 1));
#pragma unroll
  for (int g = 0; g < GROUPS; ++g) {
    const int c = 4 * (tl + 32 * g);
    if (c < 32 * nks) O::store4(ldsX + e * XP + O::off(c), pre[g][0], pre[g][1], pre[g][2], pre[g][3]);
  }
  for (int c = 4 * (tl + 32 * GROUPS); c < 32 * nks; c += 4 * 32) {
    const f32x4 v = group(c);
    O::store4(ldsX + e * XP + O::off(c), v[0], v[1], v[2], v[3]);
  }
  __syncthreads();

  f32x4 bias[FT];
  auto request_bias = [&](const float *b) {
#pragma unroll
    for (int c = 0; c < FT; ++c) bias[c] = *reinterpret_cast<const f32x4 *>(b + 16 * (ft0 + c) + 4 * q4);
  };
  static_assert(PD % Sums<BF16>::CH == 0, "");
  Sums<BF16> acc[FT];
  auto multiply = [&](const Block(&b)[FT], const unsigned char *xk, int chain) {
    Block v;
    fetch_x(v, xk);
#pragma unroll
    for (int c = 0; c < FT; ++c) mma16(b[c], v, acc[c].hi[chain], acc[c].lo);
  };
  auto put_hidden = [&](unsigned char *H) {
#pragma unroll
    for (int c = 0; c < FT; ++c) {
      f32x4 v = acc[c].total();
      v += bias[c];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = BF16 ? tanh_from_scaled(v[i] * kTwoLog2e) : tanh_accurate(v[i]);
      if (active) O::template store4<true>(H + row * HP + O::off(16 * (ft0 + c) + 4 * q4), v[0], v[1], v[2], v[3]);
      acc[c] = Sums<BF16>{};
    }
  };

  // -- layer 1
  const unsigned char *xop = ldsX + row * XP + O::off(8 * q4);
  request_bias(net.b[0]);
  int i = 0;
  const int last = nks - 1;  // (its second half may lie behind the last block: zeros there, whatever was read)
  for (; i + PD <= last; i += PD) {
#pragma unroll
    for (int s = 0; s < PD; ++s) {
      multiply(ring[s], xop + 2 * (i + s) * O::KBYTES, s % Sums<BF16>::CH);
      request(ring[s], net.W[0], nkb, min(i + s + PD, last));
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int s = 0; s < PD; ++s) {
    if (i + s < last) multiply(ring[s], xop + 2 * (i + s) * O::KBYTES, s % Sums<BF16>::CH);
    if (i + s == last) {
#pragma unroll
      for (int c = 0; c < FT; ++c)
        if (2 * last + (q4 >> 1) >= nkb) ring[s][c] = Block{};
      multiply(ring[s], xop + 2 * last * O::KBYTES, s % Sums<BF16>::CH);
    }
  }
  // -- layer 2
#pragma unroll
  for (int s = 0; s < PD && s < KS; ++s) request(ring[s], net.W[1], 2 * KS, s);
  put_hidden(ldsH1);
  request_bias(net.b[1]);
  __syncthreads();
  const unsigned char *h1op = ldsH1 + row * HP + O::off(8 * q4), *h2op = ldsH2 + row * HP + O::off(8 * q4);
#pragma unroll
  for (int k = 0; k < KS; ++k) {
    multiply(ring[k % PD], h1op + 2 * k * O::KBYTES, k % Sums<BF16>::CH);
    if (k + PD < KS) request(ring[k % PD], net.W[1], 2 * KS, k + PD);
    __builtin_amdgcn_sched_barrier(0);
  }
  // -- output layer: a tile of 16 outputs and a part of the inputs to a wavefront
  const int out = net.out_dim, ot = w & 1, kp = w >> 1;
  const bool mine = kp < KP && 16 * ot < out;
  Block w3[PER];
#pragma unroll
  for (int p = 0; p < PER; ++p)
    fetch_w(w3[p], net.W[2] + (size_t)(2 * (min(kp, KP - 1) * PER + p) + (q4 >> 1)) * NP + ot * 16 + row + 32 * (q4 & 1));
  put_hidden(ldsH2);
  __syncthreads();
  if (mine) {
    Sums<BF16> s;
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      Block v;
      fetch_x(v, h2op + 2 * (kp * PER + p) * O::KBYTES);
      mma16(w3[p], v, s.hi[p % Sums<BF16>::CH], s.lo);
    }
    *reinterpret_cast<f32x4 *>(part + (kp * kRows + row) * kPartPitch + 16 * ot + 4 * q4) = s.total();
  }
  __syncthreads();
  if (tl < out && row0 + e < a.rows) {
    float z = 0.0f;
#pragma unroll
    for (int p = 0; p < KP; ++p) z += part[(p * kRows + e) * kPartPitch + tl];
    a.Y[(row0 + e) * out + tl] = finish_out(z, net.b[2][tl], net.out_tanh);
  }
}

template <bool BF16, int HD, int PD>
hipError_t launch_inst(hipStream_t st, const QueryArgs &a) {
  constexpr auto kern = query_kernel<BF16, HD, PD>;
  const hipError_t e = allow_full_lds<kern>();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)((a.rows + kRows - 1) / kRows)), dim3(kThreads), query_lds<BF16>(HD, (a.net.nkb[0] + 1) / 2), st, a);
  return hipGetLastError();
}

}  // namespace

// Sixteen rows to a workgroup: 4096 are a round of one per compute unit, which takes as long as one workgroup, and with two
// rounds it is still the faster one.  Beyond, kernels that share a weight between more rows take over.  us a call, a launch
// per layer (or whatever served the rows) -> this; 301 inputs, 30 outputs:
//   rows            48           1024         4096         8192         16384
//   fp32,  64    13.0 ->  7.9  13.6 ->  8.6  13.2 ->  9.3  17.4 -> 14.4  27.7 -> 26.7
//   fp32, 256    14.3 -> 12.0  14.2 -> 12.6  23.0 -> 13.7  38.9 -> 24.4  40.3 -> 46.5
//   bf16, 256    13.1 ->  7.5  12.8 ->  7.9  16.0 ->  7.6  24.8 -> 11.2  20.8 -> 18.8
//   bf16, 512    13.4 -> 10.8  14.8 -> 11.3  25.0 -> 11.7  32.4 -> 21.2  28.1 -> 39.4
// Several agents: an agent's workgroups stand on one XCD, so its weights cross from memory once (xcd_run; taken as they come, four
// XCDs fetched the same 0.9 MB: 64 agents of 64 rows 23.7 -> 34 us).  us a call, a launch per layer -> this:
//   agents x rows      8 x 64         32 x 64        64 x 64        4 x 1024
//   fp32, 128       10.8 ->  7.6   12.0 ->  7.7   15.2 ->  8.0   13.9 ->  8.1
//   fp32, 256       12.0 -> 11.6   17.4 -> 12.2   23.9 -> 15.0   22.7 -> 12.1
//   bf16, 512       10.8 -> 10.1   18.9 -> 10.6   27.4 -> 13.1   24.1 -> 10.6
// A second round of workgroups with few fp32 inputs is slower than tiles of 32 or 64 rows, whose weights are read less often: 5000
// rows, critic and actor, this -> those: 64 units, 41 inputs 9.9 -> 8.6 and 9.9 -> 9.1, 121 inputs 10.3 -> 9.7 and 10.5 -> 10.2, 181
// 10.9 -> 11.4; 128 units, 41 inputs 11.5 -> 10.7 and 11.6 -> 11.2, 91 inputs 11.8 -> 11.4 and 11.9 -> 12.3, 121 12.1 -> 12.4.
// Several agents' line was drawn at 4096 rows before that; 8192 rows of 8 agents, fp32 with 256 units, would be 23 us for 41, and are not
// taken yet.  fp32 with 512 units is 2.6 MB of weights a workgroup; more than 32 outputs would be more tiles than wavefronts.
bool query_supported(int64_t rows, int S, int hidden, int outputs, int bf16, int32_t N, int32_t envs_per_agent) {
  if (hidden != 64 && hidden != 128 && hidden != 256 && !(bf16 && hidden == 512)) return false;
  if (outputs > kMaxOut || S > 640 || (envs_per_agent < N && envs_per_agent % kRows != 0)) return false;
  if (rows > 4096 && !bf16 && (hidden == 64 ? S <= 128 : hidden == 128 && S <= 96)) return false;
  return rows <= (envs_per_agent < N ? 4096 : 8192);
}

// Weights of a megabyte or more take longer through one compute unit than three launches that spread them over many, until those
// have to read them again for many rows.  us a call, a launch per layer -> this; single rows, and 4 agents of 64:
//   rows                  1             24            200           1024          1500         4 x 64
//   fp32, 256, 361  11.3 -> 11.3  12.8 -> 11.6  13.9 -> 11.9  13.1 -> 12.0  16.1 -> 12.0
//   fp32, 256, 421  11.0 -> 12.5  12.7 -> 12.9  13.6 -> 13.2  12.8 -> 13.3  16.4 -> 13.3  12.4 -> 13.1
//   fp32, 256, 601  12.2 -> 14.2  13.6 -> 14.8  14.6 -> 15.1  13.7 -> 15.2  18.1 -> 15.2  13.4 -> 15.0
//   bf16, 512, 481  10.8 -> 11.0  12.1 -> 11.4  13.0 -> 11.6   (16 rows 11.5 -> 11.3; a rollout's step of one env 15.0 -> 15.9)
//   bf16, 512, 541  10.8 -> 11.1  11.8 -> 11.6  12.6 -> 11.9
//   bf16, 512, 601  10.8 -> 12.4  12.4 -> 12.6  13.4 -> 13.0  15.0 -> 13.1  20.4 -> 13.1  12.0 -> 12.8
// (the third column: inputs; more agents share no weights: 16 x 64 rows of 601 inputs 18.0 -> 15.2 and 15.1 -> 13.1)
bool query_outweighed(int64_t rows, int S, int hidden, int bf16, bool several) {
  if (several) return rows <= 256 && S > (bf16 ? 512 : 384) && hidden == (bf16 ? 512 : 256);
  return bf16 ? hidden == 512 && S > 384 && rows < (S > 512 ? 32 : 16) : hidden == 256 && S > 384 && rows <= 1024;
}

hipError_t launch_query(hipStream_t st, const PackedNet &net, int64_t rows, const float *X, int64_t ldx, float *Y, int32_t N,
                        int32_t envs_per_agent) {
  const QueryArgs a{X, ldx, rows, net, N, envs_per_agent, Y};
  switch (net.out_dim[0]) {
    case 64: return net.bf16 ? launch_inst<true, 64, 8>(st, a) : launch_inst<false, 64, 8>(st, a);
    case 128: return net.bf16 ? launch_inst<true, 128, 8>(st, a) : launch_inst<false, 128, 8>(st, a);
    case 256: return net.bf16 ? launch_inst<true, 256, 8>(st, a) : launch_inst<false, 256, 4>(st, a);
    case 512: return launch_inst<true, 512, 6>(st, a);
  }
  return hipErrorInvalidValue;
}

}  // namespace pod
