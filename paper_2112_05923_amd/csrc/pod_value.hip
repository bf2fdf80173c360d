// The fp32 value head with 256 hidden units over a long buffer: critic values of a
// whole rollout (the critic of Sec. 4.1 and 4.2 of the paper).
#include "pod_internal.h"
#include "pod_stream.h"

namespace pod {

namespace {

using namespace stream;

// Bound by the matrix cores and the power they draw: with random numbers in all operands the chip runs this kernel at
// 1.65-1.75 GHz, the matrix pipe busy 66-69 % of the cycles (profiles/pmc_fp32_kernels.txt); with zeros it takes 8.4 us
// where it takes 11.5, without the tanh work and all but the first LDS reads of a chunk 10.1.  A workgroup takes 128 rows of
// one agent at a time (pod_stream.h); the rows' own inputs come straight from memory into the registers of the lanes that
// multiply them, two k-blocks ahead.
// 301 inputs, per 32 rows and compute unit, against 64-row tiles shared by eight wavefronts that keep taking the next one:
// 8.5 million rows of 64 agents 14.1 -> 11.9 us, 2.1 million of one agent 13.9 -> 11.7.
// 21 registers spill (88 bytes a lane), at a tile's ends and between its layers: none in the loop of layer 1, the one place
// that counts requests, where one behind the copies would lengthen the wait and not shorten it.
struct ValueRowsArgs {
  const float *X;  // rows x S, dense
  float *Y;
  PackedNet net;
  int64_t agent_rows;    // rows of an agent
  uint32_t agent_tiles;  // tiles of an agent (128 rows, the last one perhaps fewer)
  uint32_t tiles;        // of all agents
  uint32_t runs;         // an agent has 32 * runs rows in every step_rows rows
  int32_t step_rows;
  int32_t S;
};

__global__ __launch_bounds__(kThreads, 2) void value_rows_kernel(ValueRowsArgs a) {
  extern __shared__ __align__(16) unsigned char lds[];
  float *ldsB = reinterpret_cast<float *>(lds + 2 * kChunk);  // b1 | b2 | w3 | b3
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 31, g = lane >> 5;
  const uint32_t lane16 = lane * 16, part = w * kPart;
  const unsigned char *wlane = lds + operand_lane(lane) * 16;
  const int S = a.S, nkb = a.net.nkb[0];
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
  auto load_x = [&](int kb, float (&x)[8]) {
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
  // values 2 pair, 2 pair + 1 of k-block kb
  auto input_pair = [&](int kb, const float (&x)[8], int pair, Blk3 &o) {
    float u = x[2 * pair], v = x[2 * pair + 1];
    if (16 * kb + 16 > S) {
      const int c0 = 16 * kb + 8 * g + 2 * pair;
      u = c0 < S ? u : 0.0f, v = c0 + 1 < S ? v : 0.0f;
    }
    operand_pair<false>(o, pair, u, v);
  };
  const unsigned char *W1, *W2;
  auto weights = [&](int agent) {
    W1 = static_cast<const unsigned char *>(a.net.W[0]) + (size_t)agent * a.net.w_stride[0];
    W2 = static_cast<const unsigned char *>(a.net.W[1]) + (size_t)agent * a.net.w_stride[1];
  };
  auto copy1 = [&](int kb) { copy_part(W1 + (size_t)kb * kChunk + part, (cur ^ kChunk) + part, lane16); };
  // two k-blocks of half the features of layer 2
  auto copy2 = [&](int half, int kp) {
    copy_part(W2 + (size_t)((2 * kp + (w >> 1)) * 8 + 4 * half) * kBlock + (w & 1) * kPart, (cur ^ kChunk) + part, lane16);
  };
  auto stage = [&](int agent) {
    const Net net = net_of(a.net, agent);
    int i = threadIdx.x;
    asm volatile("" : "+v"(i));  // (or every address in here is kept in registers across the tiles)
    {
      ldsB[i] = net.b[0][i];
      ldsB[256 + i] = net.b[1][i];
      // output weight of hidden feature i: the parts of lane 32 g, element e of block kb
      const __bf16 *wp = reinterpret_cast<const __bf16 *>(net.W[2] + (size_t)(i >> 4) * 192 + 32 * ((i >> 3) & 1)) + (i & 7);
      ldsB[512 + i] = (float)wp[0] + ((float)wp[512] + (float)wp[1024]);
    }
    if (i == 0) ldsB[768] = net.b[2][0];
  };

  auto seek = [&](int64_t row, int there) { xrow = a.X + row * S + min(r, there - 1) * S + 8 * g; };

  uint32_t t = blockIdx.x;
  if (t >= a.tiles) return;
  int agent = agent_of(t), there, own;
  int64_t row = rows_of(t, there, own);
  seek(row, there);
  weights(agent);
  stage(agent);
  cur = kChunk;  // (the copy goes to the buffer that is not in use)
  copy1(0);
  cur = 0;
  float xa[8], xb[8];
  load_x(0, xa);
  if (nkb > 1) load_x(1, xb);
  chunk_end<0>();

  for (; t < a.tiles; t += gridDim.x) {
    const uint32_t tn = t + gridDim.x;
    const bool more = tn < a.tiles;
    f32x16 h[8];
#pragma unroll
    for (int c = 0; c < 8; ++c)
#pragma unroll
      for (int i = 0; i < 16; ++i) h[c][i] = ldsB[32 * c + 16 * (i >> 3) + 8 * g + (i & 7)];
    // ---- layer 1: a k-block per chunk; the next one's operand is formed in its last blocks
    Blk3 xo;
#pragma unroll
    for (int i = 0; i < 4; ++i) input_pair(0, xa, i, xo);
    auto layer1 = [&](int kb, float (&x)[8], const float (&xnext)[8]) {
      if (kb + 1 < nkb) copy1(kb + 1);
      else copy2(0, 0);
      if (kb + 2 < nkb) load_x(kb + 2, x);
      Blk3 xn;
      chunk_products(wlane + cur, [&](int b) -> f32x16 & { return h[b]; }, [&](int) -> const Blk3 & { return xo; },
                     [&](int b) {
                       if (b >= 6) {
                         input_pair(kb + 1, xnext, 2 * b - 12, xn);
                         input_pair(kb + 1, xnext, 2 * b - 11, xn);
                       }
                     });
      xo = xn;
      if (kb + 2 < nkb) chunk_end<2>();
      else chunk_end<0>();
      cur ^= kChunk;
    };
    for (int kb = 0; kb < nkb; kb += 2) {
      layer1(kb, xa, xb);
      if (kb + 1 < nkb) layer1(kb + 1, xb, xa);
    }
    // ---- layer 2 in two halves of its features, two k-blocks per chunk, and the output layer's dot product
    const int64_t row_now = row;
    const bool own_now = r < own;
    float y = 0.0f;
    // values 2 pair, 2 pair + 1 of k-block kb, activated the first time
    auto hidden_pair = [&](int half, int kb, int pair, Blk3 &o) {
      const int c = kb >> 1, i = 8 * (kb & 1) + 2 * pair;
      if (half == 0) {
        h[c][i] = tanh_accurate(h[c][i]);
        h[c][i + 1] = tanh_accurate(h[c][i + 1]);
      }
      operand_pair<true>(o, pair, h[c][i], h[c][i + 1]);
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) hidden_pair(0, 0, i, xo);
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      f32x16 z[4];
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int i = 0; i < 16; ++i) z[c][i] = ldsB[256 + 128 * half + 32 * c + 16 * (i >> 3) + 8 * g + (i & 7)];
#pragma unroll
      for (int kp = 0; kp < 8; ++kp) {
        if (kp < 7) {
          copy2(half, kp + 1);
        } else if (half == 0) {
          copy2(1, 0);
        } else if (more) {
          weights(agent_of(tn));
          copy1(0);
          row = rows_of(tn, there, own);
          seek(row, there);
          load_x(0, xa);
          if (nkb > 1) load_x(1, xb);
        }
        Blk3 xn[2];
        chunk_products(wlane + cur, [&](int b) -> f32x16 & { return z[b & 3]; },
                       [&](int b) -> const Blk3 & { return b < 4 ? xo : xn[0]; },
                       [&](int b) {
                         const int kb = 2 * kp + (b >> 2) + 1;
                         if (kb < 16) hidden_pair(half, kb, b & 3, xn[b >> 2]);
                         else if (half == 0) hidden_pair(1, 0, b & 3, xn[b >> 2]);
                       });
        xo = xn[1];
        // (opaque: the parts are formed again in the second half, 192 registers would hold them)
        asm volatile("" : "+v"(h[kp]));
        chunk_end<0>();
        cur ^= kChunk;
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        float part = 0.0f;  // (sixteen terms at a time: one sum over 128 leaves a larger error)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          part = fmaf(tanh_accurate(z[c][i]), ldsB[512 + 128 * half + 32 * c + 16 * (i >> 3) + 8 * g + (i & 7)], part);
          if ((i & 7) == 7) asm volatile("" : "+v"(part));  // (here, not sunk below the next half)
        }
        y += part;
      }
    }
    y += __shfl_xor(y, 32);
    if (g == 0 && own_now) __builtin_nontemporal_store(y + ldsB[768], &a.Y[row_now + r]);
    if (more && agent_of(tn) != agent) {
      agent = agent_of(tn);
      __syncthreads();  // (every wavefront has read the biases and output weights)
      stage(agent);
      __syncthreads();
    }
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
  const size_t lds = 2 * kChunk + (3 * kHidden + 32) * 4;
  const unsigned blocks = a.tiles < 2u * cus ? a.tiles : 2u * cus;
  hipLaunchKernelGGL(value_rows_kernel, dim3(blocks), dim3(kThreads), lds, st, a);
  return hipGetLastError();
}

}  // namespace pod
