// One network layer per launch for the fewest rows of networks that pod_query.hip does not take (fp32 with 512 hidden units, 1024,
// many inputs or outputs, few rows for a megabyte of weights): a policy asked for actions on a handful of observations, the steps of a few hundred envs.
//
// A kernel that carries a row tile through the network streams every weight through one compute unit: 8 MB of bf16 weights of 3001
// inputs and 1024 hidden units would take 55 us at 150 GB/s.  Here a workgroup owns 32 output features of one layer and 32
// or 64 rows and its eight wavefronts split the inputs: a launch is a memory round trip or two, a few matrix instructions
// and one exchange of partial sums through LDS.  Nothing is staged: a lane's operand is eight consecutive columns of one
// row, read from where they are.
// What bounds it is that round trip and the start of a launch; with many rows it is the rows, read again by every feature
// tile's workgroup.
#include "pod_internal.h"

#include "pod_tile.h"

namespace pod {

namespace {

using tile::f32x16;
using tile::f32x4;
using tile::u32x2;
using tile::u32x4;
typedef f32x4 f32x4u __attribute__((aligned(4)));  // rows of any width

constexpr int kWaves = 8, kThreads = 64 * kWaves;
constexpr int kPitch = 36;  // floats per row of a plane of partial sums

struct RowsArgs {
  const void *X;       // fp32 rows, or the bf16 activations of the layer before
  int64_t ldx;         // elements
  int64_t rows;
  void *Y;
  int64_t ldy;
  const void *W;       // packed weights of the layer, agent-major
  const float *b;      // padded biases, agent-major
  int64_t w_stride;    // bytes between agents
  int32_t b_stride;    // floats between agents
  int32_t in_dim, out_dim, nkb, nct;
  int32_t out_tanh;
  int32_t N, envs_per_agent;
};

enum Layer { FIRST, HIDDEN, LAST };

// Eight columns of a row as a matrix operand.  FIRST: columns from `in_dim` on are zeros (their weights are too, but what
// lies behind a row may be anything).
template <bool BF16, Layer L>
__device__ inline void load_x(float (&v)[8], u32x4 &raw, const void *row, int col, int in_dim) {
  if constexpr (BF16 && L != FIRST) {
    raw = *reinterpret_cast<const u32x4 *>(static_cast<const uint16_t *>(row) + col);
  } else {
    const float *p = static_cast<const float *>(row);
    if (L != FIRST || ((col & ~15) + 16) <= in_dim) {  // (uniform: a wavefront's lanes are in one k-block)
      const f32x4 lo = *reinterpret_cast<const f32x4u *>(p + col), hi = *reinterpret_cast<const f32x4u *>(p + col + 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = lo[i], v[4 + i] = hi[i];
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float x = p[min(col + i, in_dim - 1)];
        v[i] = col + i < in_dim ? x : 0.0f;
      }
    }
  }
}

template <bool BF16, Layer L>
__device__ inline void operand_of(u32x4 &x, const float (&v)[8], const u32x4 &raw) {
  if constexpr (L != FIRST) {
    x = raw;
  } else {
    bf16x8 o;
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = (__bf16)v[i];
    x = __builtin_bit_cast(u32x4, o);
  }
}
template <bool BF16, Layer L>
__device__ inline void operand_of(tile::Blk3 &x, const float (&v)[8], const u32x4 &) {
  bf16x8 o[3];
  split3<L != FIRST>(v, o);
#pragma unroll
  for (int i = 0; i < 3; ++i) x.p[i] = __builtin_bit_cast(u32x4, o[i]);
}

// RT: 32-row tiles per workgroup; KB: k-blocks a wavefront requests at a time.  What hides a round trip is the other
// workgroups of the compute unit rather than requests in flight, so the registers stay few: twice these blocks took 12.6
// us where this takes 11.5 (48 rows x 512 units, bf16), 14.9 where 12.6 (48 x 256, fp32), 17.4 where 15.3 (4096 x 256,
// bf16), four times these 24.3 -> 36.8 (4096 x 256, fp32).
template <bool BF16, int RT, Layer L>
__global__ __launch_bounds__(kThreads, 2) void rows_layer_kernel(RowsArgs a) {
  using O = tile::Op<BF16>;
  using Block = typename O::Block;
  constexpr int KB = RT == 1 ? 2 : 1;
  extern __shared__ __align__(16) float planes[];  // [kWaves][32 RT][kPitch]
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t row0 = (int64_t)blockIdx.x * (32 * RT);
  const int ct = blockIdx.y;
  const int agent = (int)((row0 % a.N) / a.envs_per_agent);
  const u32x4 *W = reinterpret_cast<const u32x4 *>(static_cast<const unsigned char *>(a.W) + (size_t)agent * a.w_stride) +
                   (size_t)ct * (64 * tile::kPlanes<Block>) + lane;
  constexpr int ESZ = BF16 && L != FIRST ? 2 : 4;
  const unsigned char *xrow[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t)
    xrow[t] = static_cast<const unsigned char *>(a.X) + (size_t)min(row0 + 32 * t + (lane & 31), a.rows - 1) * a.ldx * ESZ;

  f32x16 acc[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[t][i] = 0.0f;
  // wavefront w: every eighth k-block (those past the last are the last block again, times zero weights)
  for (int kb0 = w; kb0 < a.nkb; kb0 += kWaves * KB) {
    Block wt[KB];
    float v[KB][RT][8];
    u32x4 raw[KB][RT];
#pragma unroll
    for (int i = 0; i < KB; ++i) {
      const int kb = kb0 + kWaves * i;
      wt[i] = Block{};
      if (kb < a.nkb) tile::fetch_w(wt[i], W + (size_t)kb * a.nct * (64 * tile::kPlanes<Block>));
#pragma unroll
      for (int t = 0; t < RT; ++t)
        load_x<BF16, L>(v[i][t], raw[i][t], xrow[t], 16 * min(kb, a.nkb - 1) + 8 * (lane >> 5), a.in_dim);
    }
#pragma unroll
    for (int i = 0; i < KB; ++i) {
      if (kb0 + kWaves * i < a.nkb) {
#pragma unroll
        for (int t = 0; t < RT; ++t) {
          Block x;
          operand_of<BF16, L>(x, v[i][t], raw[i][t]);
          O::mma(wt[i], x, acc[t]);
        }
      }
    }
  }
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    float *p = planes + ((size_t)w * (32 * RT) + 32 * t + (lane & 31)) * kPitch + 4 * (lane >> 5);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      *reinterpret_cast<f32x4 *>(p + 8 * j) = f32x4{acc[t][4 * j], acc[t][4 * j + 1], acc[t][4 * j + 2], acc[t][4 * j + 3]};
  }
  __syncthreads();
  // four features of one row per thread
  const int r = tid >> 3, f = 4 * (tid & 7);
  if (r >= 32 * RT || row0 + r >= a.rows) return;
  f32x4 z = *reinterpret_cast<const f32x4 *>(a.b + (size_t)agent * a.b_stride + 32 * ct + f);
#pragma unroll
  for (int k = 0; k < kWaves; ++k) z += *reinterpret_cast<const f32x4 *>(planes + ((size_t)k * (32 * RT) + r) * kPitch + f);
  const int64_t at = (row0 + r) * a.ldy + 32 * ct + f;
  if constexpr (L == LAST) {
    float *Y = static_cast<float *>(a.Y) + at;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (32 * ct + f + i < a.out_dim) Y[i] = tile::finish_out(z[i], 0.0f, a.out_tanh);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) z[i] = BF16 ? tile::tanh_from_scaled(z[i] * tile::kTwoLog2e) : tile::tanh_accurate(z[i]);
    if constexpr (BF16) *reinterpret_cast<u32x2 *>(static_cast<uint16_t *>(a.Y) + at) = u32x2{bf16_pair(z[0], z[1]), bf16_pair(z[2], z[3])};
    else *reinterpret_cast<f32x4 *>(static_cast<float *>(a.Y) + at) = z;
  }
}

template <bool BF16, int RT, Layer L>
hipError_t launch_layer(hipStream_t st, const RowsArgs &a) {
  constexpr auto kern = rows_layer_kernel<BF16, RT, L>;
  const hipError_t e = allow_full_lds<kern>();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)((a.rows + 32 * RT - 1) / (32 * RT)), (unsigned)a.nct), dim3(kThreads),
                     (size_t)kWaves * 32 * RT * kPitch * 4, st, a);
  return hipGetLastError();
}

template <bool BF16, int RT>
hipError_t launch_dtype(hipStream_t st, const RowsArgs &a, int l) {
  return l == 0 ? launch_layer<BF16, RT, FIRST>(st, a) : l == 1 ? launch_layer<BF16, RT, HIDDEN>(st, a)
                                                                : launch_layer<BF16, RT, LAST>(st, a);
}

}  // namespace

// Where the lines lie, in workgroups of 64 rows x 32 features; us per forward pass, the kernels that
// take over -> this one.  A workgroup per feature tile reads the rows once each, which with many of them costs more than the
// others' staging.
//   bf16, 301 inputs: 48 rows x 512 units 28.4 -> 11.5, 1000 x 512 24.9 -> 13.6, 4096 x 256 (512 workgroups) 23.3 -> 15.3;
//   4096 x 512 (1024) 26.8 -> 30.5, 8000 x 256 25.9 -> 32.2.  1001 inputs: 1024 x 512 (256) 32.4 -> 18.1.  3001: 500 x 1024 (256)
//   55.2 -> 38.1.
//   bf16 in a rollout, whose other kernels have their rows converted already (us per step): 1024 envs x 100 stocks (256) 35.3 ->
//   29.6, 1000 x 300 x 3 indicators (256) 40.9 -> 38.1, 2000 x 60 (512) 32.1 -> 35.4; 500 stocks x 4: 256 x 1024 units (128) 52.1 ->
//   40.6, 512 x 1024 (256) 53.6 -> 54.8.
//   fp32: 8 x 512 46.9 -> 13.4, 1000 x 512 36.1 -> 20.3, 4096 x 256 28.2 -> 22.2, 4096 x 512 54.1 -> 44.2, with 1001 inputs 79.2 ->
//   70.3, with 3001 149 -> 164 and 2048 x 512 132 -> 86; 8000 x 512 88.4 -> 91.9, 8000 x 256 41.2 -> 42.3.
bool few_rows(int64_t rows, int S, int hidden, int bf16, bool converted) {
  const int64_t workgroups = (rows + 63) / 64 * (hidden / 32);
  if (!bf16) return rows <= 4096 && (S <= 1500 || workgroups <= 512);
  if (converted) return workgroups <= (S <= 2000 ? 256 : 128);
  return workgroups <= (S <= 640 ? 512 : 256);
}

namespace {
RowsArgs layer_args(const PackedNet &net, int l, int64_t rows, const void *in, int64_t ld, float *Y, int32_t N,
                    int32_t envs_per_agent) {
  RowsArgs a;
  a.X = in, a.ldx = ld, a.rows = rows;
  a.Y = l == 2 ? static_cast<void *>(Y) : net.split_h[l];
  a.ldy = l == 2 ? net.out_dim[2] : net.out_dim[0];
  a.W = net.W[l], a.b = net.b[l], a.w_stride = net.w_stride[l], a.b_stride = net.b_stride[l];
  a.in_dim = net.in_dim[l], a.out_dim = net.out_dim[l], a.nkb = net.nkb[l], a.nct = net.nct[l];
  a.out_tanh = net.out_tanh;
  a.N = N, a.envs_per_agent = envs_per_agent;
  return a;
}

// 32 rows a workgroup until every compute unit has one (2000 rows x 256 units, fp32: 17.4 us, with 64 rows 23.8), then
// 64, which halve the reads of the weights (4096 x 256: 24.1, with 32 rows 33.0)
bool two_tiles(const RowsArgs &a) { return a.rows > 32 && (a.rows + 31) / 32 * a.nct > 256; }
}  // namespace

hipError_t launch_few_rows(hipStream_t st, const PackedNet &net, int64_t rows, const float *X, int64_t ldx, float *Y,
                           int32_t N, int32_t envs_per_agent) {
  const void *in = X;
  int64_t ld = ldx;
  for (int l = 0; l < 3; ++l) {
    const RowsArgs a = layer_args(net, l, rows, in, ld, Y, N, envs_per_agent);
    hipError_t e;
    if (net.bf16) e = two_tiles(a) ? launch_dtype<true, 2>(st, a, l) : launch_dtype<true, 1>(st, a, l);
    else e = two_tiles(a) ? launch_dtype<false, 2>(st, a, l) : launch_dtype<false, 1>(st, a, l);
    if (e != hipSuccess) return e;
    in = a.Y;
    ld = a.ldy;
  }
  return hipSuccess;
}

hipError_t launch_rows_output(hipStream_t st, const PackedNet &net, int64_t rows, const void *h, int64_t pitch, float *Y,
                              int32_t N, int32_t envs_per_agent) {
  const RowsArgs a = layer_args(net, 2, rows, h, pitch, Y, N, envs_per_agent);
  return two_tiles(a) ? launch_layer<true, 2, LAST>(st, a) : launch_layer<true, 1, LAST>(st, a);
}

}  // namespace pod
