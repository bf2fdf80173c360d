// The fp32 value head with 256 hidden units over a long buffer: critic values of a
// whole rollout (the critic of Sec. 4.1 and 4.2 of the paper).
#include <type_traits>

#include "pod_internal.h"
#include "pod_stream.h"

namespace pod {

namespace {

using namespace stream;

typedef float f32x2 __attribute__((ext_vector_type(2)));

// A workgroup takes 128 rows of one agent at a time (pod_stream.h); the rows' own inputs come straight from memory into the
// registers of the lanes that multiply them, two chunks of the weights ahead.  Bound by vector work and matrix cores together, at
// the clock the power limit leaves: per 32 rows 840 matrix instructions (46 % of the cycles at 1.76 GHz) and 7000 vector ones,
// two thirds of them the two activations, with 22 % of the wavefronts' time in waits.
// 301 inputs, per 32 rows and compute unit, against products of three bf16 parts (twice the matrix work, as much vector work to
// take an operand apart): 8.5 million rows of 64 agents 11.9 -> 8.2 us; 20480 rows 49 -> 44 us, 65536 91 -> 68; 49 inputs
// 29.7 -> 30.4 and 56 -> 46, a launch that forms the parts included.  2-norm of the error against 64 bits 2.87e-7 -> 2.56e-7
// (4096 envs of 30 stocks x 8 indicators), 2.18e-7 -> 2.05e-7 (8 x 4): half as many roundings of the accumulator.
// What it took: activations four at a time with one operation under a matrix instruction (in chains, behind the read
// of their factors, 10.7 ms for 8.5), and no spilled register: a reload waits for the copies that are under way.
struct ValueRowsArgs {
  const float *X;  // rows x S, dense
  float *Y;
  PackedNet net;
  const unsigned char *H[2];  // hidden layers in fp16 parts, and their factors
  const float *U[2];
  int64_t h_stride[2];
  int64_t agent_rows;    // rows of an agent
  uint32_t agent_tiles;  // tiles of an agent (128 rows, the last one perhaps fewer)
  uint32_t tiles;        // of all agents
  uint32_t runs;         // an agent has 32 * runs rows in every step_rows rows
  int32_t step_rows;
  int32_t S;
};

__global__ __launch_bounds__(kThreads, 2) void value_rows_kernel(ValueRowsArgs a) {
  extern __shared__ __align__(16) unsigned char lds[];
  // factors and biases of both layers by feature, output weights and bias
  float *ldsU1 = reinterpret_cast<float *>(lds + 2 * kChunk), *ldsB1 = ldsU1 + 256, *ldsU2 = ldsB1 + 256, *ldsB2 = ldsU2 + 256,
        *ldsW3 = ldsB2 + 256;
  // one base per lane, constants behind it (left alone, the compiler keeps an address for every feature)
  uint32_t feature0 = 8 * ((threadIdx.x & 63) >> 5);
  asm volatile("" : "+v"(feature0));
  const float *mine = ldsU1 + feature0;
  uint32_t *ldsAgain = reinterpret_cast<uint32_t *>(ldsW3 + 264);
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 31, g = lane >> 5;
  const uint32_t lane16 = lane * 16, part = w * kPart;
  const unsigned char *wlane = lds + operand_lane(lane) * 16;
  const int S = a.S, nkb = a.net.nkb[0], nch = (nkb + 1) >> 1;
  uint32_t cur = 0;  // the chunk buffer in use

  // a tile's agent, and the first of this wavefront's 32 rows (which lie next to each other) with how many there are
  // (behind the agent's last run: that one again, and no row is the wavefront's own)
  auto agent_of = [&](uint32_t t) { return (int)(t / a.agent_tiles); };
  auto rows_of = [&](uint32_t t, int &there, int &own) {
    const uint32_t agent = t / a.agent_tiles, run0 = (t - agent * a.agent_tiles) * kWaves + w, last = (uint32_t)((a.agent_rows - 1) / 32);
    const uint32_t run = min(run0, last), step = run / a.runs, in_step = run - step * a.runs;
    there = run < last ? 32 : (int)(a.agent_rows - 32 * (int64_t)last);
    own = run0 > last ? 0 : there;
    return (int64_t)step * a.step_rows + 32 * ((int64_t)agent * a.runs + in_step);
  };
  const float *xrow;
  auto load_block = [&](int kb, float *x) {
    const float *p = xrow + 16 * kb;
    if (16 * kb + 16 <= S) {
      typedef f32x4 f32x4u __attribute__((aligned(4)));
      const f32x4 lo = *reinterpret_cast<const f32x4u *>(p), hi = *reinterpret_cast<const f32x4u *>(p + 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = lo[i], x[4 + i] = hi[i];
    } else {
      int c0 = 16 * kb + 8 * g;
      asm volatile("" : "+v"(c0));
#pragma unroll
      for (int i = 0; i < 8; ++i) x[i] = p[min(c0 + i, S - 1) - c0];
    }
  };
  // inputs of chunk ch: sixteen of the row's 32 (zeros behind the last one are put in by input_pair)
  auto load_x = [&](int ch, float (&x)[16]) {
    load_block(2 * ch, x);
    load_block(2 * ch + 1, x + 8);
  };
  float scale, unscale, top;  // of the lane's row; the largest input so far
  bool exact = false;  // (see below)
  // Inputs of chunk ch as they are multiplied: zeros behind the last one, and with `exact` none that its scale would make zero.
  auto settle = [&](int ch, float (&x)[16]) {
    if (32 * ch + 32 > S || exact) {
      int c0 = 32 * ch + 8 * g;
      asm volatile("" : "+v"(c0));
      const float smallest = exact ? 0x1p-24f * unscale : 0.0f;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        x[i] = x[i] != 0.0f && fabsf(x[i]) < smallest ? __builtin_copysignf(smallest, x[i]) : x[i];
        x[i] = c0 + 16 * (i >> 3) + (i & 7) < S ? x[i] : 0.0f;
      }
    }
  };
  // values 2 p, 2 p + 1 of a chunk
  auto input_pair = [&](const float (&x)[16], int p, Blk2 (&o)[2]) {
    top = fmaxf(fmaxf(fabsf(x[2 * p]), fabsf(x[2 * p + 1])), top);
    operand_pair<false>(o[p >> 2], p & 3, x[2 * p] * scale, x[2 * p + 1] * scale);
  };
  // The row's inputs are scaled by their largest one's power of two (to 2^4 .. 2^5): the first 32 inputs' as a rule.
  auto set_scale = [&](float largest) {
    const int e = min(max((int)(__builtin_bit_cast(uint32_t, largest) >> 23), 6), 254);
    scale = __builtin_bit_cast(float, (uint32_t)(258 - e) << 23);
    unscale = __builtin_bit_cast(float, (uint32_t)(e - 4) << 23);
  };
  const unsigned char *W1, *W2;
  auto weights = [&](int agent) {
    W1 = a.H[0] + (size_t)agent * a.h_stride[0];
    W2 = a.H[1] + (size_t)agent * a.h_stride[1];
  };
  // (the last chunk of an odd number of k-blocks has one: its second half is not there)
  auto copy1 = [&](int ch) {
    if (2 * ch + 1 < nkb || w < kWaves / 2) copy_part(W1 + (size_t)ch * kChunk + part, (cur ^ kChunk) + part, lane16);
  };
  // four k-blocks of half the features of layer 2, one copied by each wavefront
  auto copy2 = [&](int half, int kq) {
    copy_part(W2 + (size_t)((4 * kq + w) * 8 + 4 * half) * kBlock, (cur ^ kChunk) + part, lane16);
  };
  auto stage = [&](int agent) {
    const Net net = net_of(a.net, agent);
    int i = threadIdx.x;
    asm volatile("" : "+v"(i));  // (or every address in here is kept in registers across the tiles)
    ldsU1[i] = a.U[0][(size_t)agent * 256 + i];
    ldsB1[i] = net.b[0][i];
    ldsU2[i] = a.U[1][(size_t)agent * 256 + i];
    ldsB2[i] = net.b[1][i];
    // output weight of hidden feature i: the parts of lane 32 g, element e of block kb
    const __bf16 *wp = reinterpret_cast<const __bf16 *>(net.W[2] + (size_t)(i >> 4) * 192 + 32 * ((i >> 3) & 1)) + (i & 7);
    ldsW3[i] = (float)wp[0] + ((float)wp[512] + (float)wp[1024]);
    if (i == 0) ldsW3[256] = net.b[2][0];
  };

  auto seek = [&](int64_t row, int there) { xrow = a.X + row * S + min(r, there - 1) * S + 8 * g; };

  uint32_t t = blockIdx.x;
  if (t >= a.tiles) return;
  int agent = agent_of(t), there, own;
  int64_t row = rows_of(t, there, own);
  seek(row, there);
  weights(agent);
  stage(agent);
  if (tid == 0) *ldsAgain = ~0u;
  cur = kChunk;  // (the copy goes to the buffer that is not in use)
  copy1(0);
  cur = 0;
  float xa[16], xb[16];
  load_x(0, xa);
  load_x(1, xb);
  chunk_end<0>();

  // A tile with a row whose first 32 inputs did not show its size (an input more than a thousand times as large behind them,
  // or infinite, or the first ones all zero) is taken a second time, `exact`, with the scales of the whole rows.
  for (uint32_t turn = 0; t < a.tiles; ++turn) {
    f32x16 h[8];
#pragma unroll
    for (int c = 0; c < 8; ++c)
#pragma unroll
      for (int i = 0; i < 16; ++i) h[c][i] = 0.0f;
    // ---- layer 1: two k-blocks per chunk; the next ones' operands are formed in its last blocks
    Blk2 xo[2];
    auto layer1 = [&](int ch, float (&x)[16], float (&xnext)[16]) {
      if (ch + 1 < nch) copy1(ch + 1);
      else copy2(0, 0);
      if (ch + 2 < nch) load_x(ch + 2, x);
      Blk2 xn[2];
      chunk_products(wlane + cur, 2 * ch + 1 < nkb, [&](int b) -> f32x16 & { return h[b & 7]; }, [&](int b) -> const Blk2 & { return xo[b >> 3]; },
                     [&](int b, int i) {
                       if (b == 8 && i == 0) settle(ch + 1, xnext);
                       if (b >= 8 && i == 1) input_pair(xnext, b - 8, xn);
                     });
      xo[0] = xn[0], xo[1] = xn[1];
      if (ch + 2 < nch) chunk_end<4>();
      else chunk_end<0>();
      cur ^= kChunk;
    };
    float first = 0.0f;  // the largest of the inputs the scale is taken from
    if (exact) {
      for (int kb = 0; kb < nkb; ++kb)
        for (int i = 0; i < 8; ++i) {
          const float x = 16 * kb + 8 * g + i < S ? fabsf(xrow[16 * kb + i]) : 0.0f;
          first = fmaxf(first, x < __builtin_inff() ? x : 0.0f);
        }
    } else {
      settle(0, xa);
#pragma unroll
      for (int i = 0; i < 16; ++i) first = fmaxf(first, fabsf(xa[i]));
    }
    first = fmaxf(first, __shfl_xor(first, 32));
    set_scale(first > 0.0f ? first : 1.0f);
    if (exact) settle(0, xa);
    top = 0.0f;
#pragma unroll
    for (int p = 0; p < 8; ++p) input_pair(xa, p, xo);
    for (int ch = 0; ch < nch; ch += 2) {
      layer1(ch, xa, xb);
      if (ch + 1 < nch) layer1(ch + 1, xb, xa);
    }
    if (__ballot(first > 0.0f ? top * scale >= 0x1p15f : top > 0.0f) != 0 && lane == 0) *ldsAgain = turn;
    // ---- layer 2 in two halves of its features, four k-blocks per chunk, and the output layer's dot product
    const int64_t row_now = row;
    const bool own_now = r < own;
    bool again = false, more = false;
    uint32_t tn = t;
    float y = 0.0f;
    // Four values (4 q .. 4 q + 3 of the lane's eight of k-block kb): activated, scaled and taken apart, a step of it over all four
    // at a time under each of six matrix instructions.
    f32x4 u, bias;
    auto request_four = [&](int kb, int q) {
      const float *f = mine + 16 * kb + 4 * q;
      u = *reinterpret_cast<const f32x4 *>(f), bias = *reinterpret_cast<const f32x4 *>(f + 256);
    };
    float v[4], e[4], v2[4], ps[4];
    auto activate_four = [&](int step, int kb, int q, Blk2 &o) {
      f32x16 &hc = h[kb >> 1];
      const int i0 = 8 * (kb & 1) + 4 * q;
      auto all = [&](auto op) {
#pragma unroll
        for (int i = 0; i < 4; ++i) op(i);
      };
      if (step == 0) {
        all([&](int i) { v[i] = hc[i0 + i] * unscale; });
        all([&](int i) { v[i] = fmaf(v[i], u[i], bias[i]); });
        all([&](int i) { e[i] = fabsf(v[i]) * kTwoLog2e; });
        if (2 * kb + q < 31) request_four(kb + q, 1 - q);
      } else if (step == 1) {
        all([&](int i) { e[i] = __builtin_amdgcn_exp2f(e[i]); });
        all([&](int i) { v2[i] = v[i] * v[i]; });
        all([&](int i) { ps[i] = fmaf(v2[i], 62.0f / 2835.0f, -17.0f / 315.0f); });
      } else if (step == 2) {
        all([&](int i) { e[i] = e[i] + 1.0f; });
        all([&](int i) { ps[i] = fmaf(v2[i], ps[i], 2.0f / 15.0f); });
        all([&](int i) { ps[i] = fmaf(v2[i], ps[i], -1.0f / 3.0f); });
      } else if (step == 3) {
        all([&](int i) { e[i] = __builtin_amdgcn_rcpf(e[i]); });
        all([&](int i) { v2[i] = v2[i] * v[i]; });
        all([&](int i) { ps[i] = fmaf(v2[i], ps[i], v[i]); });
      } else if (step == 4) {
        all([&](int i) { e[i] = copysignf(fmaf(e[i], -2.0f * kHiddenScale, kHiddenScale), v[i]); });
        all([&](int i) { ps[i] = ps[i] * kHiddenScale; });
        all([&](int i) { v[i] = fabsf(v[i]) < 0.25f ? ps[i] : e[i]; });
      } else {
        operand_pair<true>(o, 2 * q, v[0], v[1]);
        operand_pair<true>(o, 2 * q + 1, v[2], v[3]);
        all([&](int i) { hc[i0 + i] = v[i]; });
      }
    };
    Blk2 xs[2];
    request_four(0, 0);
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int step = 0; step < 6; ++step) activate_four(step, 0, q, xs[0]);
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      f32x16 z[4];
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int i = 0; i < 16; ++i) z[c][i] = 0.0f;
#pragma unroll
      for (int kq = 0; kq < 4; ++kq) {
        if (kq < 3) {
          copy2(half, kq + 1);
        } else if (half == 0) {
          copy2(1, 0);
        } else {
          again = !exact && (uint32_t)__builtin_amdgcn_readfirstlane(*ldsAgain) == turn;
          tn = again ? t : t + gridDim.x;
          more = tn < a.tiles;
          // (behind the last tile it is taken again: inputs that are loaded on one path only would be kept all around)
          const uint32_t next = more ? tn : t;
          weights(agent_of(next));
          copy1(0);
          row = rows_of(next, there, own);
          seek(row, there);
          load_x(0, xa);
          load_x(1, xb);
        }
        chunk_products(wlane + cur, true, [&](int b) -> f32x16 & { return z[b & 3]; },
                       [&](int b) -> const Blk2 & { return xs[(b >> 2) & 1]; },
                       [&](int b, int i) {
                         const int kb = 4 * kq + (b >> 2) + 1;
                         if (half == 0 && kb < 16) {
                           activate_four(3 * (b & 1) + i, kb, (b & 3) >> 1, xs[kb & 1]);
                         } else if (i == 1 && (kb < 16 || half == 0)) {  // (once more, from the values kept)
                           const f32x16 &hc = h[(kb & 15) >> 1];
                           const int i0 = 8 * (kb & 1) + 2 * (b & 3);
                           operand_pair<true>(xs[kb & 1], b & 3, hc[i0], hc[i0 + 1]);
                         }
                       });
        // (opaque: the parts are formed again in the second half, 128 registers would hold them)
        asm volatile("" : "+v"(h[2 * kq]), "+v"(h[2 * kq + 1]));
        chunk_end<0>();
        cur ^= kChunk;
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        float part = 0.0f;  // (sixteen terms at a time: one sum over 128 leaves a larger error)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float *f = mine + 512 + 128 * half + 32 * c + 16 * (i >> 3) + (i & 7);
          part = fmaf(tanh_accurate(fmaf(z[c][i], f[0], f[256])), f[512], part);
          if ((i & 7) == 7) asm volatile("" : "+v"(part));  // (here, not sunk below the next half)
        }
        y += part;
      }
    }
    y += __shfl_xor(y, 32);
    if (g == 0 && own_now && !again) __builtin_nontemporal_store(y + ldsW3[256], &a.Y[row_now + r]);
    if (more && agent_of(tn) != agent) {
      agent = agent_of(tn);
      __syncthreads();  // (every wavefront has read the factors, biases and output weights)
      stage(agent);
      __syncthreads();
    }
    exact = again, t = tn;
  }
}

}  // namespace

// (a wavefront's 32 rows lie next to each other)
bool value_rows_covers(int64_t rows, int32_t N, int32_t envs_per_agent) {
  return rows <= 0x7fffffffll * 32 && (envs_per_agent == N || (envs_per_agent % 32 == 0 && rows % N == 0));
}

hipError_t launch_value_rows(hipStream_t st, const PackedNet &net, int64_t rows, const float *X, float *Y, int32_t N,
                             int32_t envs_per_agent, int cus) {
  ValueRowsArgs a;
  a.X = X, a.Y = Y, a.net = net, a.S = net.in_dim[0];
  const int agents = envs_per_agent < N ? N / envs_per_agent : 1;
  a.runs = agents > 1 ? envs_per_agent / 32 : 1, a.step_rows = agents > 1 ? N : 32;
  a.agent_rows = rows / agents;
  a.agent_tiles = (uint32_t)((a.agent_rows + kRows - 1) / kRows);
  a.tiles = a.agent_tiles * agents;
  HalvesJob jobs[2];
  for (int l = 0; l < 2; ++l) {
    a.H[l] = static_cast<const unsigned char *>(net.half_w[l]), a.U[l] = net.half_u[l];
    a.h_stride[l] = halves_bytes(net.nkb[l], net.nct[l]);
    jobs[l] = {net.W[l], net.w_stride[l], net.half_w[l], a.h_stride[l], net.half_u[l], net.nkb[l], net.nct[l], l == 0 ? 0 : kHiddenExp};
  }
  hipError_t err = launch_halves(st, jobs, 2, agents);
  if (err == hipSuccess) err = allow_full_lds<value_rows_kernel>();
  if (err != hipSuccess) return err;
  const size_t lds = 2 * kChunk + (5 * kHidden + 32) * 4;
  const unsigned blocks = a.tiles < 2u * cus ? a.tiles : 2u * cus;
  hipLaunchKernelGGL(value_rows_kernel, dim3(blocks), dim3(kThreads), lds, st, a);
  return hipGetLastError();
}

}  // namespace pod
