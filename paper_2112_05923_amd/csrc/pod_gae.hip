// Generalised advantage estimation as a chunked reverse scan (implied by the
// paper's use of PPO, Sec. 5.2; see compute_gae in podrollout.h).
//
// The recurrence A_t = delta_t + c_t A_{t+1} is first-order linear, so a run of
// steps can be summarised by the pair (a, p) with A_first = a + p * A_after.
// A workgroup owns W consecutive envs; a wavefront's 64 lanes are W envs x 64 / W
// chunks of GAE_L consecutive steps.  Every lane loads its whole chunk into
// registers (all loads in flight at once), scans it locally, the chunks of a
// wavefront are composed by shuffles and those of the workgroup through LDS,
// and every lane patches its results with the advantage that comes in from the
// later chunks.  Segments of NW * 64 / W * GAE_L steps are walked from the end
// of the rollout to the start with the boundary advantage carried in a register.
//
// Bound by HBM (17 bytes per step and env).  What decides the time at a few
// thousand envs is how many workgroups there are to request it: with one env per
// lane (W = 64) 5001 envs are 79 workgroups and leave two thirds of the chip
// idle.  Narrower tiles share cache lines with their neighbours, so neighbouring
// tiles go to the same XCD (one L2) and nothing is streamed past the cache there:
// with streaming stores the half-written lines cost twice the time.  Measured at
// 1000 x 5001 (85 MB): 41 us with W = 64, 26 us with W = 32, 67 us with W = 16 and
// streaming stores, 30 us without; 512 x 4096: 16 / 10 / 9 us with W = 64 / 32 / 16.
#include "pod_internal.h"

namespace pod {

constexpr int GAE_L = 16;    // steps per lane (register resident)
constexpr int GAE_NW = 16;   // wavefronts per workgroup

// PREFETCH: the next segment's rows are requested before the current one is patched and stored (one workgroup per
// compute unit).  NTL / NTS: rows are read / written once, past the cache; worth it where a row segment is whole lines.
template <int W, bool PREFETCH, bool NTL, bool NTS>
__global__ __launch_bounds__(GAE_NW * 64) void gae_kernel(int T, int N, const float *__restrict__ reward,
                                                         const float *__restrict__ value,
                                                         const uint8_t *__restrict__ done, float gamma, float gl,
                                                         float *__restrict__ adv, float *__restrict__ ret) {
  constexpr int J = 64 / W;  // chunks per wavefront
  __shared__ float s_a[GAE_NW][W];
  __shared__ float s_p[GAE_NW][W];
  const int lane = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
  const int el = lane & (W - 1);
  const int q = w * J + lane / W;  // chunk of this lane, counted from the end of the segment
  // tiles are dealt out in runs: blocks go to the 8 XCDs in turn, and an XCD's blocks take consecutive tiles
  const int per = (int)(gridDim.x >> 3);
  const int n = ((int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3)) * W + el;
  const bool live = (unsigned)n < (unsigned)N;
  constexpr int seg = GAE_NW * J * GAE_L;
  float carry = 0.0f;  // advantage at the first step of the segment handled before (later in time)

  // chunk q of the segment ending at hi covers [c_lo, c_lo + GAE_L)
  struct Rows {
    float r[GAE_L], v[GAE_L], v_after;
    uint8_t dn[GAE_L];
  };
  auto ld = [](const auto *p) { return NTL ? __builtin_nontemporal_load(p) : *p; };
  auto st = [](float x, float *p) {
    if (NTS) __builtin_nontemporal_store(x, p);
    else *p = x;
  };
  auto load = [&](int hi, bool en, Rows &x) {
    const int c_lo = hi - (q + 1) * GAE_L;
#pragma unroll
    for (int i = 0; i < GAE_L; ++i) {
      const int t = c_lo + i;
      const bool ok = en && live && t >= 0;
      const size_t idx = (size_t)(ok ? t : 0) * N + (live ? n : 0);
      x.r[i] = ok ? ld(reward + idx) : 0.0f;
      x.v[i] = ok ? ld(value + idx) : 0.0f;
      x.dn[i] = ok ? ld(done + idx) : (uint8_t)1;
    }
    const int t = c_lo + GAE_L;  // <= T: value has T+1 rows
    x.v_after = (en && live && t >= 0) ? ld(value + (size_t)t * N + n) : 0.0f;
  };
  Rows x;
  load(T, true, x);

  for (int hi = T; hi > 0; hi -= seg) {
    const int c_lo = hi - (q + 1) * GAE_L;
    float a[GAE_L], p[GAE_L];
    // local scan, newest step first
    float a_c = 0.0f, p_c = 1.0f, v_next = x.v_after;
#pragma unroll
    for (int i = GAE_L - 1; i >= 0; --i) {
      const bool skip = (c_lo + i) < 0;  // before the start of the rollout: identity
      const float g = x.dn[i] ? 0.0f : gamma;
      const float c = x.dn[i] ? 0.0f : gl;
      const float delta = fmaf(g, v_next, x.r[i]) - x.v[i];
      a_c = skip ? a_c : fmaf(c, a_c, delta);
      p_c = skip ? p_c : c * p_c;
      a[i] = a_c;
      p[i] = p_c;
      v_next = x.v[i];
    }
    // inclusive composition over the wavefront's chunks (later chunks are lower lanes)
#pragma unroll
    for (int o = W; o < 64; o *= 2) {
      const float a_o = __shfl_up(a_c, o), p_o = __shfl_up(p_c, o);
      if (lane >= o) {
        a_c = fmaf(p_c, a_o, a_c);
        p_c = p_c * p_o;
      }
    }
    if (lane >= 64 - W) {
      s_a[w][el] = a_c;
      s_p[w][el] = p_c;
    }
    Rows y;
    if (PREFETCH) load(hi - seg, hi - seg > 0, y);
    __syncthreads();
    // advantage just after this wavefront's chunks = later wavefronts of the segment applied to the carry
    float a_in = carry;
    for (int c = 0; c < w; ++c) a_in = fmaf(s_p[c][el], a_in, s_a[c][el]);
    float seg_first = a_in;
    for (int c = w; c < GAE_NW; ++c) seg_first = fmaf(s_p[c][el], seg_first, s_a[c][el]);
    carry = seg_first;
    if (J > 1) {  // ... and the later chunks of the wavefront
      const float a_o = __shfl_up(a_c, W), p_o = __shfl_up(p_c, W);
      if (lane >= W) a_in = fmaf(p_o, a_in, a_o);
    }
#pragma unroll
    for (int i = 0; i < GAE_L; ++i) {
      const int t = c_lo + i;
      if (live && t >= 0) {
        const float A = fmaf(p[i], a_in, a[i]);
        const size_t idx = (size_t)t * N + n;
        st(A, adv + idx);
        st(A + x.v[i], ret + idx);
      }
    }
    if (PREFETCH)
      x = y;
    else if (hi - seg > 0)
      load(hi - seg, true, x);
    __syncthreads();  // summaries are rewritten by the next segment
  }
}

template <int W, bool PREFETCH, bool NTL, bool NTS>
static hipError_t launch_gae_w(hipStream_t st, int32_t T, int32_t N, const float *reward, const float *value,
                               const uint8_t *done, float gamma, float lambda, float *adv, float *ret) {
  const unsigned tiles = (unsigned)((N + W - 1) / W);
  hipLaunchKernelGGL((gae_kernel<W, PREFETCH, NTL, NTS>), dim3((tiles + 7) / 8 * 8), dim3(GAE_NW * 64), 0, st, (int)T,
                     (int)N, reward, value, done, gamma, gamma * lambda, adv, ret);
  return hipGetLastError();
}

hipError_t launch_gae(hipStream_t st, int32_t T, int32_t N, const float *reward, const float *value,
                      const uint8_t *done, float gamma, float lambda, float *adv, float *ret) {
  // Widest tile that still gives the chip about 128 workgroups to request rows with (measured at 2048, 4096, 5001,
  // 11000 and 16384 envs).
  if (N > 8192) {
    const bool lines = N % 32 == 0;  // every row segment is whole cache lines
    if (T > GAE_NW * GAE_L)
      return lines ? launch_gae_w<64, true, true, true>(st, T, N, reward, value, done, gamma, lambda, adv, ret)
                   : launch_gae_w<64, true, true, false>(st, T, N, reward, value, done, gamma, lambda, adv, ret);
    return lines ? launch_gae_w<64, false, true, true>(st, T, N, reward, value, done, gamma, lambda, adv, ret)
                 : launch_gae_w<64, false, true, false>(st, T, N, reward, value, done, gamma, lambda, adv, ret);
  }
  if (N > 4096) return launch_gae_w<32, false, false, false>(st, T, N, reward, value, done, gamma, lambda, adv, ret);
  return launch_gae_w<16, false, false, false>(st, T, N, reward, value, done, gamma, lambda, adv, ret);
}

}  // namespace pod
