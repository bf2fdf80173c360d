// Trading performance of recorded rollouts (Sec. 5.3 "Performance metrics";
// what the evaluator of Sec. 4.2 reports next to the episodic reward):
// cumulative return, annual return and volatility, maximum drawdown, Sharpe
// and Calmar ratio of the account-value curve of the first episode of every
// env in an observation buffer.
//
// The value V_t = cash_t + sum_d h_{t,d} p_{t,d} is decoded from the
// observation (Table 1 state; the power-of-two scales divide out exactly) in
// binary64, stock order.  A workgroup owns ME envs and splits the time axis into
// MW * 64 / ME chunks, one per lane: lane = (env, chunk).  For every point of
// the chunks a wavefront stages the price and holdings runs of its 64 rows in
// LDS (one load instruction per row: half the lanes the prices, half the
// holdings), then each lane walks its own row there; a chunk is reduced to a
// small summary (Welford moments of the per-period returns, running peak, lowest
// value, lowest value-to-running-peak ratio) and the summaries are merged
// pairwise in time order:
//   moments:   Chan's pairwise update, the return across the seam added;
//   drawdown:  min over t of V_t / max_{s<=t} V_s over two consecutive spans
//              a, b is min(ratio_a, ratio_b, lowest_b / peak_a).
// Bound by HBM: 4 (1 + 2 D) bytes per (t, env) out of every S-float row, which
// is 3 or 4 cache lines of a row of 301 floats.  Rows of different envs share no
// line that is read, so a workgroup may own few envs: what it needs is that there
// are enough workgroups (with 64 envs each, 4096 envs kept 64 compute units busy).
#include "pod_internal.h"

namespace pod {
namespace {

constexpr int MW = 8;            // wavefronts per workgroup

struct Chunk {
  double mean, m2;         // of the returns r_t = V_{t+1} / V_t - 1 inside the chunk
  double peak, low;        // highest and lowest value
  double ratio;            // lowest V_t / (running peak within the chunk)
  double v_first, v_last;  // values at the chunk's first and last point (points after the episode's end left out)
  int32_t n_pts, pad;      // n_pts - 1 returns
};

// the summary of two consecutive spans
__device__ inline Chunk merged(const Chunk &a, const Chunk &b) {
  if (b.n_pts == 0) return a;  // (a span is empty only if everything after it is)
  Chunk c;
  const double na = (double)a.n_pts, nb = (double)(b.n_pts - 1), nt = na + nb;
  // the return across the seam joins span a's a.n_pts - 1 returns
  const double r = b.v_first / a.v_last - 1.0;
  const double d1 = r - a.mean;
  const double mean_a = a.mean + d1 / na;
  const double m2_a = a.m2 + d1 * (r - mean_a);
  const double d2 = b.mean - mean_a;
  c.mean = mean_a + d2 * (nb / nt);
  c.m2 = m2_a + b.m2 + d2 * d2 * (na * nb / nt);
  c.ratio = fmin(fmin(a.ratio, b.ratio), b.low / a.peak);
  c.peak = fmax(a.peak, b.peak);
  c.low = fmin(a.low, b.low);
  c.v_first = a.v_first;
  c.v_last = b.v_last;
  c.n_pts = a.n_pts + b.n_pts;
  c.pad = 0;
  return c;
}

struct MetricArgs {
  int32_t T, N, D, S;
  const float *obs;
  const uint8_t *done;
  double inv_cash, inv_price, inv_hold, periods, rf;
  double *metrics;
  int32_t *length;
};

// ME: envs per workgroup; MB: stocks staged at a time, one less than the lanes of a run (16 or 32): the lane left over
// in the first run carries the cash.
template <int ME, int MB>
__global__ __launch_bounds__(64 * MW) void metrics_kernel(MetricArgs a) {
  constexpr int RUN = MB + 1, RPI = 32 / RUN;  // rows per load instruction
  constexpr int MP = 2 * RUN + 1;              // floats per staged row (odd: lanes reading their own row hit distinct banks)
  constexpr int NC = MW * 64 / ME;             // chunks of the time axis
  extern __shared__ __align__(16) unsigned char lds[];
  // [MW][64][MP] staging floats; the chunk summaries reuse the space once the chunks are done
  float *stage_all = reinterpret_cast<float *>(lds);
  int32_t *s_first = reinterpret_cast<int32_t *>(stage_all + (size_t)MW * 64 * MP);  // [NC][ME]
  Chunk *s_chunk = reinterpret_cast<Chunk *>(lds);                                   // [NC][ME]
  const int T = a.T, N = a.N, D = a.D, S = a.S;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int e = lane & (ME - 1), ch = w * (64 / ME) + lane / ME;
  const int n0 = blockIdx.x * ME;
  const int n = n0 + e;
  const bool live = n < N;
  const int span = (T + 1 + NC - 1) / NC;  // points per chunk
  const int c0 = ch * span, c1 = min(c0 + span, T + 1);
  float *stage = stage_all + (size_t)w * 64 * MP;

  // ---- length of the first episode: first step whose done flag is set, else T
  int first = T;
  if (live) {
    for (int t0 = c0; t0 < min(c1, T); t0 += 8) {
      uint8_t f[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) f[i] = a.done[(size_t)min(t0 + i, T - 1) * N + n];
#pragma unroll
      for (int i = 7; i >= 0; --i)
        if (f[i] && t0 + i < min(c1, T)) first = min(first, t0 + i);
    }
  }
  s_first[ch * ME + e] = first;
  __syncthreads();
  int L = T;
  for (int c = 0; c < NC; ++c) L = min(L, s_first[c * ME + e]);

  // ---- summary of this lane's chunk: points c0 .. min(c1 - 1, L)
  Chunk ck = {};
  ck.ratio = 1.0;
  const int last = live ? min(c1 - 1, L) : -1;
  const double both = a.inv_hold * a.inv_price;  // (powers of two: scaling the exact product changes no bit of it)
  const int sub = lane / (2 * RUN), c = lane & (RUN - 1), hold = (lane / RUN) & 1;
  for (int i = 0; i < span; ++i) {
    const int t = c0 + i;
    if (!__any(t <= last)) break;
    double v = 0.0;
    for (int d0 = 0; d0 < D; d0 += MB) {
      const int bw = min(MB, D - d0);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // the previous block's reads are done
      // all of the block's loads are issued before the first of them is stored (one round trip per block)
      float x[64 / RPI];
      const bool is_cash = d0 == 0 && c == MB && !hold;
      const bool carries = c < bw || is_cash;
      const int col = is_cash ? 0 : 1 + hold * D + d0 + c;
#pragma unroll
      for (int rr = 0; rr < 64 / RPI; ++rr) {
        const int row = RPI * rr + sub;  // the lane whose point this is
        const int rt = w * (64 / ME) + row / ME, rn = n0 + (row & (ME - 1));
        const int tt = rt * span + i;
        const bool ok = carries && tt <= T && rn < N;
        x[rr] = ok ? __builtin_nontemporal_load(a.obs + ((size_t)tt * N + rn) * S + col) : 0.0f;
      }
#pragma unroll
      for (int rr = 0; rr < 64 / RPI; ++rr) stage[(RPI * rr + sub) * MP + (lane & (2 * RUN - 1))] = x[rr];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // LDS executes a wavefront's accesses in order
      const float *mine = stage + lane * MP;
      if (d0 == 0) v = (double)mine[MB] * a.inv_cash;
#pragma unroll 4
      for (int j = 0; j < bw; ++j) v = fma((double)mine[RUN + j] * (double)mine[j], both, v);
    }
    if (t <= last) {
      if (i == 0) {
        ck.v_first = ck.peak = ck.low = v;
      } else {
        const double r = v / ck.v_last - 1.0;
        const double dlt = r - ck.mean;
        ck.mean += dlt / (double)i;
        ck.m2 += dlt * (r - ck.mean);
        ck.peak = fmax(ck.peak, v);
        ck.low = fmin(ck.low, v);
        ck.ratio = fmin(ck.ratio, v / ck.peak);
      }
      ck.v_last = v;
      ck.n_pts = i + 1;
    }
  }
  __syncthreads();  // staging buffers are dead: the summaries go over them
  s_chunk[ch * ME + e] = ck;

  // ---- merge pairs of neighbouring spans, in time order, until one is left
  for (int half = NC / 2; half > 0; half /= 2) {
    const int step = NC / half / 2;  // chunks per span
    __syncthreads();
    for (int i = threadIdx.x; i < half * ME; i += 64 * MW) {
      const int p = i / ME, pe = i & (ME - 1);
      Chunk *s = s_chunk + (size_t)(2 * step * p) * ME + pe;
      *s = merged(*s, s[(size_t)step * ME]);
    }
  }
  __syncthreads();
  if (w == 0 && lane < ME && live) {
    const Chunk m = s_chunk[e];
    double out[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (L >= 1) {
      const double sd = L >= 2 ? sqrt(m.m2 / (double)(L - 1)) : 0.0;
      const double mdd = 1.0 - m.ratio;
      out[0] = (m.v_last - m.v_first) / m.v_first;
      out[1] = pow(m.v_last / m.v_first, a.periods / (double)L) - 1.0;
      out[2] = sqrt(a.periods) * sd;
      out[3] = mdd;
      out[4] = sd > 0.0 ? sqrt(a.periods) * (m.mean - a.rf / a.periods) / sd : 0.0;
      out[5] = mdd > 0.0 ? out[1] / mdd : 0.0;
    }
    for (int i = 0; i < 6; ++i) a.metrics[(size_t)i * N + n] = out[i];
    if (a.length) a.length[n] = L;
  }
}

template <int ME, int MB>
hipError_t launch_metrics(hipStream_t st, const MetricArgs &a) {
  size_t lds = (size_t)MW * 64 * (2 * (MB + 1) + 1) * 4;
  if (lds < (size_t)MW * 64 * sizeof(Chunk)) lds = (size_t)MW * 64 * sizeof(Chunk);
  lds += (size_t)MW * 64 * 4;
  const hipError_t e = allow_full_lds<metrics_kernel<ME, MB>>();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((metrics_kernel<ME, MB>), dim3((unsigned)((a.N + ME - 1) / ME)), dim3(64 * MW), lds, st, a);
  return hipGetLastError();
}

template <int MB>
hipError_t launch_metrics_mb(hipStream_t st, const MetricArgs &a) {
  // Few envs per workgroup, so that there are two workgroups for every compute unit, as long as the chunks of the
  // time axis keep a few points each (a chunk costs a step of the merge tree whatever its length).
  const int64_t points = a.T + 1;
  if (a.N >= 16 * 512 || points < 4 * MW * 64 / 16) {
    if (a.N >= 64 * 512 || points < 4 * MW) return launch_metrics<64, MB>(st, a);
    return launch_metrics<16, MB>(st, a);
  }
  if (a.N >= 8 * 512 || points < 4 * MW * 64 / 4) return launch_metrics<8, MB>(st, a);
  return launch_metrics<4, MB>(st, a);
}

}  // namespace

hipError_t launch_trading_metrics(hipStream_t st, int32_t T, int32_t N, int32_t D, int32_t S, const float *obs,
                                  const uint8_t *done, const float *obs_scale, double periods, double rf,
                                  double *metrics, int32_t *length) {
  MetricArgs a;
  a.T = T;
  a.N = N;
  a.D = D;
  a.S = S;
  a.obs = obs;
  a.done = done;
  a.inv_cash = 1.0 / (double)obs_scale[0];
  a.inv_price = 1.0 / (double)obs_scale[1];
  a.inv_hold = 1.0 / (double)obs_scale[2];
  a.periods = periods;
  a.rf = rf;
  a.metrics = metrics;
  a.length = length;
  return D <= 15 ? launch_metrics_mb<15>(st, a) : launch_metrics_mb<31>(st, a);
}

}  // namespace pod
