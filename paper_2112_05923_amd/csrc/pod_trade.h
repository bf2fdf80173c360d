// The trades of one env step (Table 1 and Sec. 5.3 of the paper), shared by the
// kernel that steps all envs once and the one that keeps small networks and
// their envs on a compute unit for a whole rollout.
//
// Included only by translation units that are compiled with floating-point
// contraction off: the share counts are decided by a fixed sequence of binary32
// operations with one rounding each.
#pragma once

#include "pod_internal.h"

namespace pod {
namespace {

constexpr int kEnvThreads = 512;
typedef float env_f32x4 __attribute__((ext_vector_type(4)));
typedef env_f32x4 env_f32x4u __attribute__((aligned(4)));
typedef double env_f64x2 __attribute__((ext_vector_type(2)));

struct __attribute__((aligned(16))) Purchase {
  float k, u;   // wanted shares, unit cost
  double rcp;   // 1 / u in binary64
};

__device__ inline double sum_lanes(double v, int width) {
  for (int o = 1; o < width; o *= 2) v += __shfl_xor(v, o);
  return v;
}

// Account values are the cash plus the holdings h p in stock order, in binary64.  Threads that add them up in another
// order get the same number when nothing is rounded on the way: cash and products are multiples of some 2^x, and while no
// sum exceeds 2^53 of them every partial sum is a binary64 number.  Multiples of what: a product of the last place of its
// price p, at least 2^-24 p; the cash of its lowest bit that is set (cash_unit is that or, for a power of two, less).
// `lowest`: the smallest price, negative if a holding is; the bound leaves a factor of two for the rounding of the values
// themselves, and fails for values that are negative, infinite or no numbers.
__device__ inline float cash_unit(float c) {
  const uint32_t b = __builtin_bit_cast(uint32_t, c);
  return c - __builtin_bit_cast(float, b & (b - 1));
}
__device__ inline bool order_free(double v0, double v1, float lowest, float cash0, float cash1) {
  const float bound = fminf(fminf(lowest * 0x1p28f, 0x1p127f), fminf(cash_unit(cash0), cash_unit(cash1)) * 0x1p52f);
  const float f0 = (float)v0, f1 = (float)v1;
  return f0 >= 0.0f && f1 >= 0.0f && f0 <= bound && f1 <= bound;
}

// s + v[0][0] + v[0][1] + ... in this order (two register sets, read one ahead of the other by hand, were slower)
__device__ inline float serial_sum(float s, const env_f32x4 *v, int n) {
#pragma unroll 8
  for (int c = 0; c < n; ++c) {
    const env_f32x4 x = v[c];
    s = s + x[0];
    s = s + x[1];
    s = s + x[2];
    s = s + x[3];
  }
  return s;
}

// NT threads (the workgroup's 512, or its last 256) trade for E envs: TPE = NT / E neighbouring threads own one env, and a thread the stocks tl, tl + TPE, ...
// (at most ND) of its env, whose prices, holdings and orders stay in its registers.  What bounds the step is the chain
// prices -> orders -> the serial walk over the purchases -> holdings; everything else hangs off it:
//  - the ledger adds the sales from a dense row, and walks only the purchases: the threads pack them into a list in
//    stock order (ballots inside a wavefront, counts through LDS across two).  It runs in the env's own wavefront
//    (half) and needs one dependent operation per purchase while the cash lasts, none for a purchase it does not
//    buy a single share of, and the quotient only in between (13.5 -> 1.8 us of a step with 250 purchases);
//  - the account values before and after are sums over the env's threads, taken again in stock order by one of them where
//    the order shows in the last bit (prices far apart in size).  With WALK they are always taken in stock order, by value()
//    and not here: a kernel that goes on with the same envs knows the value before and needs the one after for the reward
//    only.  Where one workgroup has the compute unit to itself the sums over lanes take longer (rollout_small_kernel, 5
//    stocks 3.97 -> 3.60 us a step, 30 stocks 5.16 -> 4.98); where others want the same issue slots it is the other way
//    round (env_step_kernel, 16384 envs x 30 stocks 15.5 us against 16.3, 4096 x 64 8.0 against 9.1);
//  - up to a wavefront per env there is no barrier in here: an env's threads only meet each other.
// The reciprocals of the unit costs (unit_of) are the caller's, before its actions are known, and with WALK so is the account
// value: rollout_small_kernel, which had both in here, 16 envs x 5 stocks 3.55 -> 3.47 us a step, 512 x 30 with 64 units 5.30
// -> 5.11, bf16 with 128 4.61 -> 4.38, fp32 with 128 level.
// SET: the kernel sets the thread's index `me`, an opaque copy of it in each step, or what follows from it is kept across them.
// (Held where nobody sets it, it costs rollout_small_kernel 2 %.)
template <int E, int ND, bool WALK, int NT = kEnvThreads, bool SET = false>
struct Trade {
  static constexpr int TPE = NT / E;
  static constexpr int CW = TPE < 64 ? TPE : 64;  // the part of a wavefront one env has
  static constexpr int NCW = TPE / CW;            // wavefronts per env
  static constexpr int CHUNK = CW < 16 ? CW : 16; // purchases tried in full together
  static_assert((!WALK || NCW == 1) && CW % CHUNK == 0 && CHUNK % 4 == 0 && (NT & (NT - 1)) == 0, "");
  int me;
  __device__ inline int thread() const { return SET ? me : threadIdx.x & (NT - 1); }
  int D, D4, lp, sp, op;
  Purchase *list;  // [E][lp] purchases in stock order (odd pitch in 16 bytes)
  float *sell;     // [E][sp] proceeds of the sales, 0 elsewhere
  float *sq;       // [E][sp] squared noise
  float *out;      // [E][op] outlay k u of the purchases, by list position
  int32_t *buy;    // [E][lp] shares bought, by list position
  double *part;    // [2][E][2] holdings' value before / after, per wavefront of an env
  float *low;      // [E][2] and their smallest price
  float *both;     // [E][2] cash before / after
  float *e2s;      // [E] sum of the squares
  int32_t *cnt;    // [E][ND NCW] purchases
  float *now;      // several wavefronts per env (whose registers are few): [E][D4] prices of the trades
  double *terms;   // WALK: [E][D4] holdings' values after the trades, in stock order

  __device__ Trade(unsigned char *lds, int D_) : me(threadIdx.x & (NT - 1)), D(D_), D4((D_ + 3) & ~3), lp(D_ | 1), sp(D4 + 4), op(D4 + 20) {
    list = reinterpret_cast<Purchase *>(lds);
    sell = reinterpret_cast<float *>(list + E * lp);
    sq = sell + E * sp;
    out = sq + E * sp;
    buy = reinterpret_cast<int32_t *>(out + E * op);
    part = reinterpret_cast<double *>(buy + E * lp);
    low = reinterpret_cast<float *>(part + 4 * E);
    both = low + 2 * E;
    e2s = both + 2 * E;
    cnt = reinterpret_cast<int32_t *>(e2s + E);
    now = reinterpret_cast<float *>(cnt + 8 * E);
    terms = reinterpret_cast<double *>(now);
  }

  // all of an env's threads have written what the others read
  __device__ static void meet() {
    if (NCW > 1) {
      __syncthreads();
    } else {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
  }

  // What a purchase of the thread's stocks needs of their prices alone (a binary64 division: where the prices are known
  // before the actions, this is too).
  struct Unit {
    float cost[ND];
    double rcp[ND];  // 1 / cost
  };
  __device__ static Unit unit_of(const EnvDims &d, const float (&pn)[ND]) {
    Unit u;
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      u.cost[i] = pn[i] * d.one_plus_c;
      u.rcp[i] = 1.0 / (double)u.cost[i];
    }
    return u;
  }

  // Sampled actions a_raw and their noise, prices pn the trades execute at and pv the account is valued at afterwards,
  // holdings h (updated), executed shares q (signed), cash (updated); e2 (the summed squares if wanted) is complete in the
  // env's first thread, and without WALK r (the reward).  market(): between sizing and ledger; rest(): behind the ledger;
  // booked(i): the thread's i-th stock is settled (live stocks only).
  template <class Market, class Rest, class Booked>
  __device__ inline void run(const EnvDims &d, bool live, const float (&a_raw)[ND], const float (&eps)[ND], const float (&pn)[ND],
                             const Unit &units, const float (&pv)[ND], int32_t (&h)[ND], int32_t (&q)[ND], float &cash, double &r,
                             float &e2, bool want_e2, Market market, Rest rest, Booked booked) {
    const int tid = thread(), lane = tid & 63;
    const int e = tid / TPE, tl = tid & (TPE - 1), cw = tl / CW, cl = lane & (CW - 1);
    const float cash_in = cash;
    auto mine_of = [&](uint64_t all) {  // the env's part of a ballot
      return CW == 64 ? all : (all >> (lane & ~(CW - 1))) & ((1ull << (CW & 63)) - 1ull);
    };
    // -- size the orders
    int32_t rank[ND], total = 0;
    float kf[ND];
    double a0 = 0.0;
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      const int dd = tl + TPE * i;
      const bool ok = live && dd < D;
      const float ac = fminf(1.0f, fmaxf(-1.0f, a_raw[i]));
      const int32_t k = ok ? (int32_t)truncf(ac * d.hmax) : 0;
      float sale = 0.0f;
      q[i] = 0;
      kf[i] = 0.0f;
      if (!WALK) a0 += ok ? (double)h[i] * (double)pn[i] : 0.0;
      if (k < 0) {
        const int32_t qs = min(-k, h[i]);
        h[i] -= qs;
        const float gross = pn[i] * (float)qs;
        sale = gross * d.one_minus_c;
        q[i] = -qs;
      } else if (k > 0) {
        kf[i] = (float)k;
      }
      if (dd < D4) {
        sell[e * sp + dd] = sale;
        if (NCW > 1) now[e * D4 + dd] = pn[i];
        sq[e * sp + dd] = ok ? eps[i] * eps[i] : 0.0f;
      }
      const uint64_t mine = mine_of(__ballot(k > 0));
      rank[i] = __popcll(mine & ((1ull << cl) - 1ull));
      if (NCW == 1) {
        rank[i] += total;
        total += __popcll(mine);
      } else if (cl == 0) {
        cnt[(e * ND + i) * NCW + cw] = __popcll(mine);
      }
    }
    if (!WALK) a0 = sum_lanes(a0, CW);
    if (NCW > 1) {
      if (cl == 0) part[e * 2 + cw] = a0;
      __syncthreads();
#pragma unroll
      for (int i = 0; i < ND; ++i)
#pragma unroll
        for (int w = 0; w < NCW; ++w) {
          const int c = cnt[(e * ND + i) * NCW + w];
          if (w == cw) rank[i] += total;
          total += c;
        }
    }
#pragma unroll
    for (int i = 0; i < ND; ++i)
      if (kf[i] > 0.0f) {
        list[e * lp + rank[i]] = Purchase{kf[i], units.cost[i], units.rcp[i]};
        out[e * op + rank[i]] = kf[i] * units.cost[i];
      }
    if (tl < 16) out[e * op + total + tl] = 0.0f;
    market();
    meet();

    // the squares are summed in stock order (the log-probability is the same number in every schedule), and so are the sales
    e2 = 0.0f;
    const env_f32x4 *sales = reinterpret_cast<const env_f32x4 *>(sell + e * sp), *squares = reinterpret_cast<const env_f32x4 *>(sq + e * sp);
    if (WALK) {
#pragma unroll 4
      for (int c = 0; c < D4 / 4; ++c) {
        const env_f32x4 x = sales[c], y = squares[c];
        cash = cash + x[0], e2 = e2 + y[0];
        cash = cash + x[1], e2 = e2 + y[1];
        cash = cash + x[2], e2 = e2 + y[2];
        cash = cash + x[3], e2 = e2 + y[3];
      }
    } else if (cw == NCW - 1 && want_e2) {
      e2 = serial_sum(0.0f, squares, D4 / 4);
      if (NCW > 1 && cl == 0) e2s[e] = e2;
    }
    if (cw == 0) {
      // -- the ledger (Table 1 actions: sell / buy / hold): all sales, then all purchases, in stock order, each limited
      // by the cash left:
      //   m = floor(cash / u); q = min(k, max(m, 0)); if (q u > cash) q -= 1; cash -= q u        (binary32)
      if (!WALK) cash = serial_sum(cash, sales, D4 / 4);
      const Purchase *lst = list + e * lp;
      auto affordable = [&](float c, float u) { return mine_of(__ballot(!(c < u))); };
      for (int c0 = 0; c0 < total; c0 += CW) {
        const int p = c0 + cl;
        const Purchase mine = lst[min(p, total - 1)];
        const float u = p < total ? mine.u : __builtin_inff();
        int32_t got = 0;
        constexpr uint64_t all = (1ull << CHUNK) - 1ull;
        for (int s0 = 0; s0 < CW && c0 + s0 < total; s0 += CHUNK) {
          if (((affordable(cash, u) >> s0) & all) == 0) continue;
          // sixteen (or eight) purchases in full: as long as the balance stays clear of 0 (2^-20 of what it was, so every outlay
          // k u before it was below the balance by more than its own rounding), each quotient was at least k
          const env_f32x4 *ov = reinterpret_cast<const env_f32x4 *>(out + e * op + c0 + s0);
          const float clear = cash * 0x1p-20f;
          float full = cash;
          int in_full = 0;
#pragma unroll
          for (int c = 0; c < CHUNK / 4; ++c) {
            const env_f32x4 v = ov[c];
            full = full - v[0];
            full = full - v[1];
            full = full - v[2];
            full = full - v[3];
            if (full >= clear) cash = full, in_full = 4 * c + 4;  // (outlays are not negative: never true again once false)
          }
          if ((unsigned)(cl - s0) < (unsigned)in_full) got = (int32_t)mine.k;
          if (in_full == CHUNK) continue;
          // one by one, those that buy nothing (cash < u: the quotient is below 1 and rounds below 1) skipped.
          // The binary32 quotient comes from one binary64 product with the prepared reciprocal of u: the product is
          // within 2^-52 of cash / u, and a quotient of two binary32 numbers is at least 2^-49 (relative) away from
          // every binary32 rounding boundary it does not hit exactly, so the product rounded to binary32 is the
          // correctly rounded cash / u.  It is never negative (cash is not), so truncation is the floor and needs no
          // clamp at 0; the outlay of one share less, (q - 1) u rounded once, is the fused q u - u.
          uint64_t ahead = (all << s0) & (~0ull << (s0 + in_full));
          while (true) {
            const uint64_t left = affordable(cash, u) & ahead;
            if (left == 0) break;
            const int j = __builtin_ctzll(left);
            const Purchase b = lst[c0 + j];
            const float ratio = (float)((double)cash * b.rcp);
            const float q0 = fminf(b.k, truncf(ratio));
            const float out_q = q0 * b.u, out_q1 = fmaf(q0, b.u, -b.u);
            const float bal0 = cash - out_q, bal1 = cash - out_q1;
            const bool over = out_q > cash;
            cash = over ? bal1 : bal0;
            if (cl == j) got = (int32_t)(over ? q0 - 1.0f : q0);
            ahead &= ~1ull << j;
          }
        }
        if (p < total) buy[e * lp + p] = got;
      }
    }
    rest();
    meet();

    // -- executed trades, holdings, account value after them
    double a1 = 0.0, v0 = (double)cash_in, v1 = (double)cash;
    float lowest = __builtin_inff();
    int32_t sign = 0;
    int32_t h1[ND];
    // (not WALK) the values' terms in stock order where the purchases were, which all of an env's threads are past
    double *term0 = reinterpret_cast<double *>(list + e * lp), *term1 = term0 + lp;
    auto price_now = [&](int i) { return NCW > 1 ? now[e * D4 + min(tl + TPE * i, D - 1)] : pn[i]; };
    auto put_terms = [&](int i) {
      const int dd = tl + TPE * i;
      if (dd < D) term0[dd] = (double)(h1[i] - q[i]) * (double)price_now(i), term1[dd] = (double)h1[i] * (double)pv[i];
    };
    auto add_terms = [&]() {
      v0 = (double)cash_in, v1 = (double)cash;
#pragma unroll 8
      for (int dd = 0; dd < D; ++dd) v0 += term0[dd], v1 += term1[dd];
    };
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      const int dd = tl + TPE * i;
      if (kf[i] > 0.0f) {
        q[i] = buy[e * lp + rank[i]];
        h[i] += q[i];
      }
      h1[i] = h[i];
      const double term = (double)h[i] * (double)pv[i];
      if (WALK) put_term(i, dd < D ? term : 0.0);
      if (live && dd < D) {
        a1 += term;
        if (!WALK) lowest = fminf(lowest, fminf(price_now(i), pv[i])), sign |= h[i] | (h[i] - q[i]);
        booked(i);
      }
    }
    if (!WALK) {
      a1 = sum_lanes(a1, CW);
      if (sign < 0) lowest = -1.0f;
      bool again;  // for the whole workgroup, or wavefront
      if (NCW > 1) {
        for (int o = 1; o < CW; o *= 2) lowest = fminf(lowest, __shfl_xor(lowest, o));
        if (cl == 0) part[2 * E + e * 2 + cw] = a1, low[e * 2 + cw] = lowest;
        if (tl == 0) both[e * 2] = cash_in, both[e * 2 + 1] = cash;
        __syncthreads();
        // every wavefront looks at all envs: they agree without another barrier
        const int el = lane & (E - 1);
        double w0 = (double)both[el * 2], w1 = (double)both[el * 2 + 1];
        lowest = __builtin_inff();
#pragma unroll
        for (int w = 0; w < NCW; ++w)
          w0 += part[el * 2 + w], w1 += part[2 * E + el * 2 + w], lowest = fminf(lowest, low[el * 2 + w]);
        again = __ballot(!order_free(w0, w1, lowest, both[el * 2], both[el * 2 + 1])) != 0;
        v0 = __shfl(w0, e), v1 = __shfl(w1, e);
        e2 = e2s[e];
      } else {
        v0 += a0;
        v1 += a1;
        again = __ballot(live && !order_free(v0, v1, lowest, cash_in, cash)) != 0;
      }
      if (again) {
#pragma unroll
        for (int i = 0; i < ND; ++i) put_terms(i);
        meet();
        if (tl == 0) add_terms();
      }
      r = (v1 - v0) * (double)d.rho;
    }
  }

  // WALK: the account value after run(), in stock order (all of an env's threads take it)
  __device__ inline double value(float cash) const {
    const env_f64x2 *t = reinterpret_cast<const env_f64x2 *>(terms + (thread() / TPE) * D4);
    double v = (double)cash;
    meet();
#pragma unroll 4
    for (int c = 0; c < D4 / 2; ++c) {
      const env_f64x2 x = t[c];
      v = v + x[0];
      v = v + x[1];
    }
    return v;
  }
  __device__ inline void put_term(int i, double term) {  // of the thread's i-th stock, of the D4
    const int t = thread(), dd = (t & (TPE - 1)) + TPE * i;
    if (dd < D4) terms[(t / TPE) * D4 + dd] = term;
  }
};

inline size_t trade_lds(int E, bool walk, int D) {
  const int D4 = (D + 3) & ~3, lp = D | 1;
  return (size_t)E * lp * sizeof(Purchase) + (size_t)E * (2 * (D4 + 4) + D4 + 20) * 4 + (size_t)E * lp * 4 +
         (size_t)4 * E * 8 + (size_t)4 * E * 4 + (size_t)E * 4 + (size_t)E * 8 * 4 +
         (walk ? (size_t)E * D4 * 8 : E * 64 < kEnvThreads ? (size_t)E * D4 * 4 : 0);
}

}  // namespace
}  // namespace pod
