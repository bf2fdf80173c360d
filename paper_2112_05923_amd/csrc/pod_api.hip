// C ABI of libpodrollout: argument validation, workspace layout and the
// sequencing of kernel launches.  No arithmetic of the method lives here.
#include <math.h>

#include <algorithm>
#include <new>
#include <pthread.h>
#include <stdlib.h>
#include <string.h>

#include "pod_internal.h"

using namespace pod;

struct pr_handle {
  pr_config cfg;
  hipStream_t stream;
  EnvDims dims;
  EnvState st;
  pr_market market;
  PackedNet actor, critic;
  PackedNet actor_rot;    // the actor with layer 1 packed for inputs in the order [indicators | cash | prices | holdings],
                          // or [indicators | prices | holdings | cash] (market_first)
  void *w1_rot;           // (null when no rollout of this handle reads that order)
  PackedNet critic_rot;   // the critic likewise, where its hidden layers run beside the actor's (null W[0]: they do not)
  void *beside_h[2];      // its activations: of one step, and of `beside_steps` steps
  int32_t beside_steps;
  void *w_packed[2][3];   // device, per net and layer
  float *b_packed[2][3];
  float *mu_scratch;      // [N, D]
  int32_t *start;         // [N] episode start rows (zeros unless a replay table is set)
  ObsShadow shadow;       // bf16 observations of the layer-per-launch actor, or null
  void *split[3];         // hidden activations and input of the layer-per-launch networks (small batches) of a rollout
  void *query[3];         // the same for rollout_mlp_forward, whose launches for one call are enqueued under `enqueue`
  pthread_mutex_t enqueue;
  int32_t table_rows;     // rows of the market
  void *table_w[2][2];    // shared tables: layer 1 of either network, market and portfolio part (null: another schedule)
  float *table_p;         // and its sums over market rows
  int32_t *tau0;          // [N] cursors at the start of a rollout
  int32_t S;
};

namespace {

thread_local int g_last_hip = 0;

int hip_fail(hipError_t e) {
  g_last_hip = (int)e;
  return PR_EHIP;
}

#define POD_HIP(call)                       \
  do {                                      \
    hipError_t e__ = (call);                \
    if (e__ != hipSuccess) return hip_fail(e__); \
  } while (0)

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

bool is_pow2_float(float x) {
  if (!(x > 0.0f) || isinf(x)) return false;
  int e;
  return frexpf(x, &e) == 0.5f;
}

struct Layout {
  size_t w[2][3], b[2][3];
  size_t w1_rot, w1_beside, beside_h[2];
  size_t cash, tau, h, ep_ret, ep_sum, ep_sqsum, ep_cnt, mu, start, split[3], query[3];
  size_t table_w[2][2], table_p, tau0;
  size_t total;
};

int state_dim(const pr_config &c) { return 1 + 2 * c.n_stocks + c.n_stocks * c.n_ind; }

// the stepwise policy of small bf16 batches reads a bf16 copy of the observations, written along with them
bool uses_shadow(const pr_config &c) {
  return c.schedule == PR_SCHED_STEPWISE && !small_supported(c) && !table_supported(c) && layers_supported(c.n_envs, c.hidden, c.mlp_dtype) &&
         !few_rows(c.n_envs, state_dim(c), c.hidden, c.mlp_dtype, true) &&
         !query_supported(c.n_envs, state_dim(c), c.hidden, c.n_stocks, c.mlp_dtype, c.n_envs, c.n_envs / c.n_agents);
}

// rollouts of this config read layer 1 in the order [indicators | cash | prices | holdings]
bool uses_rotated(const pr_config &c) { return c.schedule == PR_SCHED_FUSED || small_supported(c) || uses_shadow(c); }

// The value head's hidden layers run beside the actor's, step by step, on the bf16 rows the actor reads, instead of over the whole
// record afterwards, where that fills compute units the actor's leave idle (or one round of taller tiles) and the inputs are too
// many for the kernels that keep a tile's inputs in LDS.  Rollouts, us per step: 2048 envs x 300 stocks, 512 units 53.3 -> 48.2,
// 1024 x 300 with 1024 units 52.1 -> 46.3, 600 x 500 56.5 -> 51.5, 1500 x 130, 512 units 35.7 -> 33.8.  One round of tall
// tiles, 1665 to 2048 rows with 1024 units: 2048 x 500 82.2 -> 78.5, 1700 x 500 80.0 -> 76.1, 2048 x 300 67.6 -> 65.9, 1800 x 300 x 3
// 64.6 -> 62.1, level at 150 stocks (50.8; 1700 x 150 x 2 47.0 -> 47.4).  With more tiles than that
// it is slower: 1400 x 200 with 1024 units (352 tiles) 50.9 -> 52.9, 4000 x 100, 512 units (504) 48.8 -> 51.6.
bool value_beside(const pr_config &c) { return uses_shadow(c) && state_dim(c) > 320 && layers_room_beside(c.n_envs, c.n_envs / c.n_agents, c.hidden); }
// steps whose last activations are kept for one launch of the output layer: 32 MiB, or one step's
int32_t value_beside_steps(const pr_config &c) {
  const int64_t step = (int64_t)c.n_envs * layers_pitch(c.hidden) * 2;
  return (int32_t)std::max<int64_t>(1, ((int64_t)32 << 20) / step);
}

// k-blocks of that copy of layer 1.  The persistent fp32 rollout of few envs reads blocks of 32 inputs, with the cash last,
// so that all market columns come first.
bool market_first(const pr_config &c) { return c.schedule == PR_SCHED_FUSED && c.mlp_dtype == PR_MLP_F32; }
int rotated_blocks(const pr_config &c) {
  const int nkb = (state_dim(c) + 15) / 16;
  return market_first(c) ? (nkb + 1) & ~1 : nkb;
}

// k-blocks of the market (0) and the portfolio (1) part of layer 1 in rollouts over a shared table
int table_blocks(const pr_config &c, int part) {
  return part == 0 ? table_market_blocks(c.n_stocks, c.n_ind) : table_portfolio_blocks(c.n_stocks);
}

int validate_config(const pr_config *c) {
  if (!c) return PR_EINVAL;
  if (c->n_envs < 1 || c->n_agents < 1 || c->n_envs % c->n_agents != 0) return PR_EINVAL;
  if (c->n_stocks < 1 || c->n_ind < 0 || c->hidden < 1 || c->horizon < 1) return PR_EINVAL;
  if (c->n_market != 1 && c->n_market != c->n_envs) return PR_EINVAL;
  if (c->mlp_dtype != PR_MLP_F32 && c->mlp_dtype != PR_MLP_BF16) return PR_EINVAL;
  if (c->schedule != PR_SCHED_STEPWISE && c->schedule != PR_SCHED_FUSED) return PR_EINVAL;
  if (!(c->cash0 > 0.0f) || !(c->hmax > 0.0f) || !(c->cost >= 0.0f) || !(c->cost < 1.0f)) return PR_EINVAL;
  if (!(c->sigma > 0.0f) || !isfinite(c->reward_scale) || !isfinite(c->cash0) || !isfinite(c->hmax)) return PR_EINVAL;
  for (int i = 0; i < 4; ++i)
    if (!is_pow2_float(c->obs_scale[i])) return PR_EINVAL;
  // index arithmetic inside the kernels is 32-bit per step and per market row
  const double nd = (double)c->n_envs * c->n_stocks * (c->n_ind > 1 ? c->n_ind : 1);
  const double rows = ((double)c->horizon + 1.0) * c->n_market;
  if (nd >= 2147483647.0 || rows >= 2147483647.0 || (double)c->n_envs * state_dim(*c) >= 2147483647.0)
    return PR_EINVAL;
  // shapes the kernels cover
  const int S = state_dim(*c);
  if (!mlp_supported(S, c->hidden, c->n_stocks, c->mlp_dtype) || !mlp_supported(S, c->hidden, 1, c->mlp_dtype))
    return PR_EUNSUPPORTED;
  if (c->n_agents > 1 && (c->n_envs / c->n_agents) % 64 != 0) return PR_EUNSUPPORTED;
  if (c->schedule == PR_SCHED_FUSED && !fused_supported(*c)) return PR_EUNSUPPORTED;
  return PR_OK;
}

Layout make_layout(const pr_config &c) {
  Layout L;
  const int S = state_dim(c), Hd = c.hidden, D = c.n_stocks, P = c.n_agents, bf = c.mlp_dtype;
  const size_t N = (size_t)c.n_envs;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = align_up(off + bytes, 256);
    return o;
  };
  const int in_dim[3] = {S, Hd, Hd};
  for (int net = 0; net < 2; ++net) {
    const int out_dim[3] = {Hd, Hd, net == 0 ? D : 1};
    for (int l = 0; l < 3; ++l) {
      L.w[net][l] = take(packed_weight_bytes(in_dim[l], out_dim[l], bf) * P);
      L.b[net][l] = take((size_t)padded_out(out_dim[l]) * 4 * P);
    }
  }
  L.w1_rot = uses_rotated(c) ? take(packed_weight_bytes(16 * rotated_blocks(c), Hd, bf) * P) : 0;
  L.w1_beside = L.beside_h[0] = L.beside_h[1] = 0;
  if (value_beside(c)) {
    L.w1_beside = take(packed_weight_bytes(16 * rotated_blocks(c), Hd, bf) * P);
    L.beside_h[0] = take(N * layers_pitch(Hd) * 2);
    L.beside_h[1] = take(value_beside_steps(c) * N * layers_pitch(Hd) * 2);
  }
  L.cash = take(N * 4);
  L.tau = take(N * 4);
  L.h = take(N * D * 4);
  L.ep_ret = take(N * 8);
  L.ep_sum = take(N * 8);
  L.ep_sqsum = take(N * 8);
  L.ep_cnt = take(N * 4);
  L.mu = take(N * D * 4);
  L.start = take(N * 4);
  const size_t rows = (size_t)split_scratch_rows(c.n_envs, Hd);
  for (size_t *scratch : {L.split, L.query}) {
    for (int i = 0; i < 2; ++i) scratch[i] = take(bf ? rows * layers_pitch(Hd) * 2 : rows * Hd * 4);
    scratch[2] = take(bf ? rows * layers_pitch(S) * 2 : 0);
  }
  if (table_supported(c)) {
    for (int net = 0; net < 2; ++net)
      for (int part = 0; part < 2; ++part) L.table_w[net][part] = take(packed_weight_bytes(16 * table_blocks(c, part), Hd, bf));
    L.table_p = take(table_scratch_bytes(c.n_envs, c.horizon));
    L.tau0 = take(N * 4);
  }
  L.total = off;
  return L;
}

// scratch of the layer-per-launch paths; null: only kernels that need none
void set_scratch(PackedNet &pn, void *const *scratch) {
  const bool any = scratch && pn.split_rows;
  for (int i = 0; i < 2; ++i) pn.split_h[i] = any ? scratch[i] : nullptr;
  pn.split_x.p = any && pn.bf16 ? static_cast<uint16_t *>(scratch[2]) : nullptr;
}

// Work enqueued now may run beside what the handle's stream does later: a graph can be replayed on any stream, and the
// per-thread stream is another one for each thread.
bool leaves_the_stream(hipStream_t st) {
  if (st == hipStreamPerThread) return true;
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &capture) == hipSuccess) return capture != hipStreamCaptureStatusNone;
  (void)hipGetLastError();  // (asked of the default stream while another one is captured)
  return true;
}

void fill_net(PackedNet &pn, const pr_handle *h, int net) {
  const pr_config &c = h->cfg;
  const int S = h->S, Hd = c.hidden, D = c.n_stocks, bf = c.mlp_dtype;
  const int in_dim[3] = {S, Hd, Hd};
  const int out_dim[3] = {Hd, Hd, net == 0 ? D : 1};
  for (int l = 0; l < 3; ++l) {
    pn.W[l] = h->w_packed[net][l];
    pn.b[l] = h->b_packed[net][l];
    pn.w_stride[l] = (int64_t)packed_weight_bytes(in_dim[l], out_dim[l], bf);
    pn.b_stride[l] = padded_out(out_dim[l]);
    pn.in_dim[l] = in_dim[l];
    pn.out_dim[l] = out_dim[l];
    pn.nkb[l] = (in_dim[l] + 15) / 16;
    pn.nct[l] = (out_dim[l] + 31) / 32;
  }
  pn.bf16 = bf;
  pn.out_tanh = net == 0 ? 1 : 0;
  pn.split_rows = split_scratch_rows(c.n_envs, Hd);
  set_scratch(pn, h->split);
  pn.split_x.pitch = layers_pitch(S);
  pn.split_x.cols = (S + 15) / 16 * 16;
}

bool weights_ok(const pr_weights *w) { return w && w->W1 && w->b1 && w->W2 && w->b2 && w->W3 && w->b3; }

int pack_nets(pr_handle *h, const pr_weights *actor, const pr_weights *critic) {
  const pr_config &c = h->cfg;
  const int S = h->S, Hd = c.hidden, D = c.n_stocks, P = c.n_agents, bf = c.mlp_dtype;
  const pr_weights *ws[2] = {actor, critic};
  PackJob jobs[kMaxPackJobs];
  int n = 0;
  for (int net = 0; net < 2; ++net) {
    const float *W[3] = {ws[net]->W1, ws[net]->W2, ws[net]->W3};
    const float *b[3] = {ws[net]->b1, ws[net]->b2, ws[net]->b3};
    const int in_dim[3] = {S, Hd, Hd};
    const int out_dim[3] = {Hd, Hd, net == 0 ? D : 1};
    for (int l = 0; l < 3; ++l)
      jobs[n++] = {W[l], b[l], h->w_packed[net][l], h->b_packed[net][l], in_dim[l], out_dim[l], (in_dim[l] + 15) / 16, {{0, 0, in_dim[l]}}};
  }
  // The persistent rollout kernel keeps its observation tile as [indicators | cash | prices | holdings] (and so do
  // the one for small networks and the bf16 copy of the observations): the same layer-1 weights with their rows rotated
  // by the D K indicator columns (biases are shared).
  const int DK = D * c.n_ind;
  if (h->w1_rot) {
    const int cash = market_first(c) ? 1 : 0;  // the cash behind the others, or in front of them
    PackJob &j = jobs[n++] = {actor->W1, actor->b1, h->w1_rot, h->b_packed[0][0], S, Hd, rotated_blocks(c),
                              {{0, 1 + 2 * D, DK}, {DK, cash, 1 + 2 * D - cash}, {S - cash, 0, cash}}};
    if (h->critic_rot.W[0]) {
      PackJob &k = jobs[n++] = j;
      k.W = critic->W1, k.b = critic->b1, k.Wp = const_cast<void *>(h->critic_rot.W[0]), k.bp = h->b_packed[1][0];
    }
  }
  // Over a shared table layer 1 is taken in two parts: [indicators | prices], and [holdings | zeros | cash].
  for (int net = 0; net < 2 && h->table_w[0][0]; ++net) {
    jobs[n++] = {ws[net]->W1, ws[net]->b1, h->table_w[net][0], h->b_packed[net][0], S, Hd, table_blocks(c, 0),
                 {{0, 1 + 2 * D, DK}, {(DK + 3) & ~3, 1, D}}};
    jobs[n++] = {ws[net]->W1, ws[net]->b1, h->table_w[net][1], h->b_packed[net][0], S, Hd, table_blocks(c, 1),
                 {{0, 1 + D, D}, {16 * table_blocks(c, 1) - 1, 0, 1}}};
  }
  POD_HIP(launch_pack_layers(h->stream, jobs, n, P, bf));
  return PR_OK;
}

int check_buffers(const pr_buffers *o) {
  if (!o || !o->obs || !o->act_raw || !o->reward || !o->done) return PR_EINVAL;
  return PR_OK;
}

TableNet table_net(const pr_handle *h, int net) {
  TableNet t;
  t.Wm = h->table_w[net][0], t.Wp = h->table_w[net][1];
  for (int l = 0; l < 3; ++l) t.W[l] = h->w_packed[net][l], t.b[l] = h->b_packed[net][l];
  return t;
}

StepIO step_io(const pr_handle *h, const pr_buffers *o, int t, const float *mu, const float *noise, const ObsShadow &shadow) {
  const size_t N = (size_t)h->cfg.n_envs, D = (size_t)h->cfg.n_stocks, S = (size_t)h->S;
  StepIO io;
  io.mu = mu;
  io.noise = noise + (size_t)t * N * D;
  io.obs_next = o->obs + (size_t)(t + 1) * N * S;
  io.act_raw = o->act_raw + (size_t)t * N * D;
  io.reward = o->reward + (size_t)t * N;
  io.done = o->done + (size_t)t * N;
  io.logp = o->logp ? o->logp + (size_t)t * N : nullptr;
  io.shadow = shadow;
  io.ind_done = false;
  io.shares = o->shares ? o->shares + (size_t)t * N * D : nullptr;
  return io;
}

}  // namespace

extern "C" {

int rollout_workspace_bytes(const pr_config *cfg, size_t *out) {
  if (!out) return PR_EINVAL;
  const int rc = validate_config(cfg);
  if (rc != PR_OK) return rc;
  *out = make_layout(*cfg).total;
  return PR_OK;
}

int rollout_kernel_lds_bytes(const pr_config *cfg, int32_t with_actor, size_t *out) {
  if (!out || !cfg) return PR_EINVAL;
  pr_config c = *cfg;
  c.schedule = PR_SCHED_STEPWISE;  // (validate the shape itself; whether the persistent kernel covers it is asked below)
  const int rc = validate_config(&c);
  if (rc != PR_OK) return rc;
  if (!fused_supported(*cfg)) return PR_EUNSUPPORTED;
  *out = fused_lds_bytes(*cfg, with_actor != 0);
  return PR_OK;
}

int rollout_init(const pr_config *cfg, const pr_market *market, const pr_weights *actor, const pr_weights *critic,
                 void *workspace, size_t workspace_bytes, void *hip_stream, pr_handle **out) {
  if (!out) return PR_EINVAL;
  *out = nullptr;
  const int rc = validate_config(cfg);
  if (rc != PR_OK) return rc;
  if (!market || !market->price || (cfg->n_ind > 0 && !market->ind)) return PR_EINVAL;
  if (!weights_ok(actor) || !weights_ok(critic)) return PR_EINVAL;
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u)) return PR_EINVAL;
  // the persistent kernel moves indicator rows in 16-byte groups
  if (cfg->schedule == PR_SCHED_FUSED && (reinterpret_cast<uintptr_t>(market->ind) & 15u)) return PR_EINVAL;
  const Layout L = make_layout(*cfg);
  if (workspace_bytes < L.total) return PR_ENOMEM;

  pr_handle *h = new (std::nothrow) pr_handle;
  if (!h) return PR_ENOMEM;
  memset(h, 0, sizeof(*h));
  if (pthread_mutex_init(&h->enqueue, nullptr) != 0) {
    delete h;
    return PR_ENOMEM;
  }
  h->cfg = *cfg;
  h->stream = static_cast<hipStream_t>(hip_stream);
  h->market = *market;
  h->S = state_dim(*cfg);
  unsigned char *ws = static_cast<unsigned char *>(workspace);
  for (int net = 0; net < 2; ++net)
    for (int l = 0; l < 3; ++l) {
      h->w_packed[net][l] = ws + L.w[net][l];
      h->b_packed[net][l] = reinterpret_cast<float *>(ws + L.b[net][l]);
    }
  h->st.cash = reinterpret_cast<float *>(ws + L.cash);
  h->st.tau = reinterpret_cast<int32_t *>(ws + L.tau);
  h->st.h = reinterpret_cast<int32_t *>(ws + L.h);
  h->st.ep_ret = reinterpret_cast<double *>(ws + L.ep_ret);
  h->st.ep_sum = reinterpret_cast<double *>(ws + L.ep_sum);
  h->st.ep_sqsum = reinterpret_cast<double *>(ws + L.ep_sqsum);
  h->st.ep_cnt = reinterpret_cast<int32_t *>(ws + L.ep_cnt);
  h->mu_scratch = reinterpret_cast<float *>(ws + L.mu);
  h->start = reinterpret_cast<int32_t *>(ws + L.start);
  for (int i = 0; i < 3; ++i) h->split[i] = ws + L.split[i], h->query[i] = ws + L.query[i];
  h->st.start = h->start;
  h->table_rows = cfg->horizon + 1;
  if (table_supported(*cfg)) {
    for (int net = 0; net < 2; ++net)
      for (int part = 0; part < 2; ++part) h->table_w[net][part] = ws + L.table_w[net][part];
    h->table_p = reinterpret_cast<float *>(ws + L.table_p);
    h->tau0 = reinterpret_cast<int32_t *>(ws + L.tau0);
  }

  EnvDims &d = h->dims;
  d.N = cfg->n_envs;
  d.D = cfg->n_stocks;
  d.K = cfg->n_ind;
  d.S = h->S;
  d.H = cfg->horizon;
  d.M = cfg->n_market;
  d.cash0 = cfg->cash0;
  d.hmax = cfg->hmax;
  d.one_minus_c = 1.0f - cfg->cost;
  d.one_plus_c = 1.0f + cfg->cost;
  d.sigma = cfg->sigma;
  d.rho = cfg->reward_scale;
  d.logp_const = (float)(-(double)cfg->n_stocks * (log((double)cfg->sigma) + 0.91893853320467274178));
  d.s_cash = cfg->obs_scale[0];
  d.s_price = cfg->obs_scale[1];
  d.s_hold = cfg->obs_scale[2];
  d.s_ind = cfg->obs_scale[3];

  fill_net(h->actor, h, 0);
  h->w1_rot = uses_rotated(*cfg) ? static_cast<void *>(ws + L.w1_rot) : nullptr;
  h->actor_rot = h->actor;
  h->actor_rot.W[0] = h->w1_rot;
  h->actor_rot.nkb[0] = rotated_blocks(*cfg);
  h->actor_rot.w_stride[0] = (int64_t)packed_weight_bytes(16 * rotated_blocks(*cfg), cfg->hidden, cfg->mlp_dtype);
  fill_net(h->critic, h, 1);
  if (uses_shadow(*cfg)) h->shadow = h->actor.split_x;
  if (value_beside(*cfg)) {
    h->critic_rot = h->critic;
    h->critic_rot.W[0] = ws + L.w1_beside;
    h->critic_rot.nkb[0] = h->actor_rot.nkb[0], h->critic_rot.w_stride[0] = h->actor_rot.w_stride[0];
    for (int i = 0; i < 2; ++i) h->beside_h[i] = ws + L.beside_h[i];
    h->beside_steps = value_beside_steps(*cfg);
  }
  int prc = pack_nets(h, actor, critic);
  if (prc == PR_OK) {
    hipError_t e = hipMemsetAsync(h->start, 0, (size_t)cfg->n_envs * 4, h->stream);
    if (e == hipSuccess) e = launch_state_reset(h->stream, h->dims, h->st);
    if (e != hipSuccess) prc = hip_fail(e);
  }
  if (prc != PR_OK) {
    rollout_destroy(h);
    return prc;
  }
  *out = h;
  return PR_OK;
}

int rollout_set_weights(pr_handle *h, const pr_weights *actor, const pr_weights *critic) {
  if (!h || !weights_ok(actor) || !weights_ok(critic)) return PR_EINVAL;
  return pack_nets(h, actor, critic);
}

int rollout_reset(pr_handle *h) {
  if (!h) return PR_EINVAL;
  POD_HIP(launch_state_reset(h->stream, h->dims, h->st));
  return PR_OK;
}

int rollout_set_replay(pr_handle *h, const pr_market *table, int32_t table_rows, const int32_t *start) {
  if (!h || !table || !table->price || (h->cfg.n_ind > 0 && !table->ind) || !start) return PR_EINVAL;
  if (table_rows < h->cfg.horizon + 1 || (double)table_rows * h->cfg.n_market >= 2147483647.0) return PR_EINVAL;
  if (h->cfg.schedule == PR_SCHED_FUSED && (reinterpret_cast<uintptr_t>(table->ind) & 15u)) return PR_EINVAL;
  // every episode must stay inside the table: checked on the device, read back here (this call synchronises)
  int32_t *flag = reinterpret_cast<int32_t *>(h->mu_scratch), bad = 1;
  POD_HIP(launch_check_starts(h->stream, h->cfg.n_envs, h->cfg.horizon, table_rows, start, flag));
  POD_HIP(hipMemcpyAsync(&bad, flag, sizeof(bad), hipMemcpyDeviceToHost, h->stream));
  POD_HIP(hipStreamSynchronize(h->stream));
  if (bad) return PR_EINVAL;
  POD_HIP(hipMemcpyAsync(h->start, start, (size_t)h->cfg.n_envs * 4, hipMemcpyDeviceToDevice, h->stream));
  h->market = *table;
  h->table_rows = table_rows;
  POD_HIP(launch_state_reset(h->stream, h->dims, h->st));
  return PR_OK;
}

int rollout_step_T(pr_handle *h, int32_t T, const float *noise, const pr_buffers *out) {
  if (!h || T < 1 || !noise) return PR_EINVAL;
  int rc = check_buffers(out);
  if (rc != PR_OK) return rc;
  const size_t N = (size_t)h->cfg.n_envs, D = (size_t)h->cfg.n_stocks, S = (size_t)h->S;
  const int32_t per_agent = h->cfg.n_envs / h->cfg.n_agents;
  if (h->table_p) {
    const TableMarket m{h->market.price, h->market.ind, h->table_rows};
    POD_HIP(launch_rollout_table(h->stream, h->dims, h->st, m, table_net(h, 0), h->table_p, h->tau0, T, noise, *out, compute_units()));
    const int64_t rows = (int64_t)(T + 1) * (int64_t)N;
    if (out->value && value_table_covers(rows, h->S, (int32_t)N, h->cfg.horizon, h->table_rows)) {
      POD_HIP(launch_value_table(h->stream, h->dims, h->st, m, table_net(h, 1), h->table_p, h->tau0, rows, out->obs, out->value,
                                 compute_units()));
      return PR_OK;
    }
  } else if (h->cfg.schedule == PR_SCHED_FUSED) {
    POD_HIP(launch_rollout_fused(h->stream, h->cfg, h->dims, h->st, h->market.price, h->market.ind, h->actor_rot,
                                 per_agent, T, noise, nullptr, *out));
  } else if (small_supported(h->cfg)) {
    POD_HIP(launch_rollout_small(h->stream, h->dims, h->st, h->market.price, h->market.ind, h->actor_rot, per_agent, T, noise,
                                 *out));
    const int64_t rows = (int64_t)(T + 1) * (int64_t)N;
    if (out->value && value_small_covers(h->critic, rows)) {
      POD_HIP(launch_value_small(h->stream, h->critic, rows, out->obs, h->S, out->value, (int32_t)N, per_agent, compute_units()));
      return PR_OK;
    }
  } else {
    POD_HIP(launch_observe(h->stream, h->dims, h->st, h->market.price, h->market.ind, out->obs, h->shadow));
    const bool beside = out->value && h->critic_rot.W[0];
    PackedNet critic = h->critic_rot;
    const size_t step_bytes = N * layers_pitch(h->cfg.hidden) * 2;
    // where the value head's activations of step t go, and its outputs once the slots are full or the record ends
    auto value_slot = [&](int t) {
      critic.split_h[0] = h->beside_h[0];
      critic.split_h[1] = static_cast<unsigned char *>(h->beside_h[1]) + (size_t)(t % h->beside_steps) * step_bytes;
    };
    auto value_out = [&](int t) {
      const int filled = t % h->beside_steps + 1;
      if (filled < h->beside_steps && t < T) return hipSuccess;
      return launch_value_dot(h->stream, critic, (int64_t)filled * (int64_t)N, h->beside_h[1], out->value + (size_t)(t + 1 - filled) * N,
                              (int32_t)N, per_agent);
    };
    for (int t = 0; t < T; ++t) {
      float *mu = out->mu ? out->mu + (size_t)t * N * D : h->mu_scratch;
      StepIO io = step_io(h, out, t, mu, noise, h->shadow);
      if (h->shadow.p) {
        if (beside) value_slot(t);
        IndicatorMove move{h->dims, h->st, h->market.ind, io.obs_next, h->shadow, false};
        POD_HIP(launch_layers(h->stream, h->actor_rot, (int64_t)N, h->shadow, mu, (int32_t)N, per_agent,
                              h->cfg.n_ind > 0 ? &move : nullptr, beside ? &critic : nullptr));
        if (beside) POD_HIP(value_out(t));
        io.ind_done = move.moved;
      } else {
        POD_HIP(launch_mlp(h->stream, h->actor, (int64_t)N, out->obs + (size_t)t * N * S, (int64_t)S, mu, (int32_t)N,
                           per_agent));
      }
      POD_HIP(launch_env_step(h->stream, h->dims, h->st, h->market.price, h->market.ind, io));
    }
    if (beside) {
      value_slot(T);
      POD_HIP(launch_hidden(h->stream, critic, (int64_t)N, h->shadow, (int32_t)N, per_agent));
      POD_HIP(value_out(T));
      return PR_OK;
    }
  }
  if (out->value)
    POD_HIP(launch_mlp(h->stream, h->critic, (int64_t)(T + 1) * (int64_t)N, out->obs, (int64_t)S, out->value,
                       (int32_t)N, per_agent));
  return PR_OK;
}

int rollout_step_forced(pr_handle *h, int32_t T, const float *mu, const float *noise, const pr_buffers *out) {
  if (!h || T < 1 || !noise || !mu) return PR_EINVAL;
  int rc = check_buffers(out);
  if (rc != PR_OK) return rc;
  const size_t N = (size_t)h->cfg.n_envs, D = (size_t)h->cfg.n_stocks;
  if (h->cfg.schedule == PR_SCHED_FUSED) {
    POD_HIP(launch_rollout_fused(h->stream, h->cfg, h->dims, h->st, h->market.price, h->market.ind,
                                 h->actor_rot, h->cfg.n_envs / h->cfg.n_agents, T, noise, mu, *out));
    return PR_OK;
  }
  POD_HIP(launch_observe(h->stream, h->dims, h->st, h->market.price, h->market.ind, out->obs, ObsShadow{}));
  for (int t = 0; t < T; ++t)
    POD_HIP(launch_env_step(h->stream, h->dims, h->st, h->market.price, h->market.ind,
                            step_io(h, out, t, mu + (size_t)t * N * D, noise, ObsShadow{})));
  return PR_OK;
}

int rollout_mlp_forward(pr_handle *h, int32_t net, int64_t rows, const float *X, int64_t ldx, float *Y) {
  if (!h || (net != PR_NET_ACTOR && net != PR_NET_CRITIC) || rows < 1 || !X || !Y || ldx < h->S) return PR_EINVAL;
  if ((rows + 63) / 64 > 2147483647LL) return PR_EINVAL;
  PackedNet pn = net == PR_NET_ACTOR ? h->actor : h->critic;
  // Queries have scratch of their own, beside a rollout's, in which the handle's stream orders them; the launches of one
  // call stay together.  A query that leaves the stream takes the kernels that keep nothing between launches, as those of
  // launch_query do anyway (8 rows x 512 units in fp32 47 us for 13).
  pthread_mutex_lock(&h->enqueue);
  set_scratch(pn, leaves_the_stream(h->stream) ? nullptr : h->query);
  const hipError_t e = launch_mlp(h->stream, pn, rows, X, ldx, Y, h->cfg.n_envs, h->cfg.n_envs / h->cfg.n_agents);
  pthread_mutex_unlock(&h->enqueue);
  POD_HIP(e);
  return PR_OK;
}

int rollout_get_state(pr_handle *h, const pr_state *out) {
  if (!h || !out) return PR_EINVAL;
  POD_HIP(launch_state_copy(h->stream, h->dims, h->st, *out, true));
  return PR_OK;
}

int rollout_set_state(pr_handle *h, const pr_state *in) {
  if (!h || !in) return PR_EINVAL;
  POD_HIP(launch_state_copy(h->stream, h->dims, h->st, *in, false));
  return PR_OK;
}

int compute_gae(void *hip_stream, int32_t T, int32_t N, const float *reward, const float *value, const uint8_t *done,
                float gamma, float lambda, float *adv, float *ret) {
  if (T < 1 || N < 1 || !reward || !value || !done || !adv || !ret) return PR_EINVAL;
  if (!isfinite(gamma) || !isfinite(lambda)) return PR_EINVAL;
  if ((double)(T + 1) * (double)N >= 9.0e18) return PR_EINVAL;
  POD_HIP(launch_gae(static_cast<hipStream_t>(hip_stream), T, N, reward, value, done, gamma, lambda, adv, ret));
  return PR_OK;
}

int trading_metrics(void *hip_stream, int32_t T, int32_t N, int32_t n_stocks, int32_t state_dim, const float *obs,
                    const uint8_t *done, const float *obs_scale, double periods_per_year, double risk_free,
                    double *metrics, int32_t *length) {
  if (T < 1 || N < 1 || n_stocks < 1 || !obs || !done || !obs_scale || !metrics) return PR_EINVAL;
  if (state_dim < 1 + 2 * n_stocks) return PR_EINVAL;
  if (!(periods_per_year > 0.0) || !isfinite(periods_per_year) || !isfinite(risk_free)) return PR_EINVAL;
  for (int i = 0; i < 3; ++i)
    if (!is_pow2_float(obs_scale[i])) return PR_EINVAL;
  if (((double)T + 1.0) * (double)N * (double)state_dim >= 9.0e18) return PR_EINVAL;
  POD_HIP(launch_trading_metrics(static_cast<hipStream_t>(hip_stream), T, N, n_stocks, state_dim, obs, done, obs_scale,
                                 periods_per_year, risk_free, metrics, length));
  return PR_OK;
}

int population_refill(void *hip_stream, int32_t P, int64_t count, const int32_t *rank, int32_t keep, float sigma,
                      const float *noise, float *params) {
  if (P < 1 || count < 1 || !rank || !params || keep < 1 || keep > P || P > 65535) return PR_EINVAL;
  if (!isfinite(sigma) || (sigma != 0.0f && !noise)) return PR_EINVAL;
  if ((double)P * (double)count >= 9.0e18) return PR_EINVAL;
  POD_HIP(launch_population_refill(static_cast<hipStream_t>(hip_stream), P, count, rank, keep, sigma,
                                   sigma != 0.0f ? noise : nullptr, params));
  return PR_OK;
}

namespace {

bool net_ok(const pr_net_params *p) { return p && p->W1 && p->b1 && p->W2 && p->b2 && p->W3 && p->b3; }

int ppo_config_ok(const pr_ppo_config *c) {
  if (!c || c->batch < 1 || c->n_stocks < 1 || c->n_ind < 0 || c->hidden < 32 || c->hidden % 32 != 0) return PR_EINVAL;
  if (!(c->sigma > 0.0f) || !(c->clip > 0.0f) || !(c->clip < 1.0f) || !(c->value_coef >= 0.0f)) return PR_EINVAL;
  if (!isfinite(c->sigma) || !isfinite(c->value_coef)) return PR_EINVAL;
  if ((double)c->batch * (double)(1 + 2 * c->n_stocks + c->n_stocks * c->n_ind) >= 2147483647.0) return PR_EINVAL;
  return PR_OK;
}

// sizes of the six tensors of a network with O outputs
void net_sizes(const pr_ppo_config &c, int O, int64_t n[6]) {
  const int64_t S = 1 + 2 * c.n_stocks + c.n_stocks * c.n_ind, Hd = c.hidden;
  n[0] = S * Hd, n[1] = Hd, n[2] = Hd * Hd, n[3] = Hd, n[4] = Hd * O, n[5] = O;
}

size_t ppo_scratch(const pr_ppo_config &c, bool adam) {
  return ppo_scratch_bytes(c.batch, c.hidden, c.n_stocks, 1 + c.n_stocks * (2 + c.n_ind), adam);
}

size_t grads_bytes(const pr_ppo_config &c) {
  int64_t a[6], b[6];
  net_sizes(c, c.n_stocks, a);
  net_sizes(c, 1, b);
  size_t t = 0;
  for (int i = 0; i < 6; ++i) t += align_up((size_t)a[i] * 4, 256) + align_up((size_t)b[i] * 4, 256);
  return t;
}

}  // namespace

int ppo_workspace_bytes(const pr_ppo_config *cfg, size_t *out) {
  if (!out) return PR_EINVAL;
  const int rc = ppo_config_ok(cfg);
  if (rc != PR_OK) return rc;
  *out = ppo_scratch(*cfg, true) + grads_bytes(*cfg);  // (gradients alone never need more)
  return PR_OK;
}

int ppo_minibatch_grads(void *hip_stream, const pr_ppo_config *cfg, const float *obs, const float *act_raw,
                        const float *logp_old, const float *adv, const float *ret, const int32_t *rows,
                        const pr_net_params *actor, const pr_net_params *critic, const pr_net_params *grad_actor,
                        const pr_net_params *grad_critic, void *workspace, size_t workspace_bytes, float *stats) {
  const int rc = ppo_config_ok(cfg);
  if (rc != PR_OK) return rc;
  if (!obs || !act_raw || !logp_old || !adv || !ret || !workspace) return PR_EINVAL;
  if (!net_ok(actor) || !net_ok(critic) || !net_ok(grad_actor) || !net_ok(grad_critic)) return PR_EINVAL;
  if ((reinterpret_cast<uintptr_t>(workspace) & 255u) ||
      workspace_bytes < ppo_scratch(*cfg, false))
    return PR_EINVAL;
  POD_HIP(launch_ppo(static_cast<hipStream_t>(hip_stream), *cfg, obs, act_raw, logp_old, adv, ret, rows, *actor, *critic,
                     *grad_actor, *grad_critic, nullptr, workspace, stats));
  return PR_OK;
}

int ppo_minibatch_grads_noalloc(void *hip_stream, const pr_ppo_config *cfg, const float *obs, const float *act_raw,
                                const float *logp_old, const float *adv, const float *ret, const int32_t *rows,
                                const pr_net_params *actor, const pr_net_params *critic,
                                const pr_net_params *grad_actor, const pr_net_params *grad_critic, float *stats) {
  const int rc = ppo_config_ok(cfg);
  if (rc != PR_OK) return rc;
  if (!obs || !act_raw || !logp_old || !adv || !ret) return PR_EINVAL;
  if (!net_ok(actor) || !net_ok(critic) || !net_ok(grad_actor) || !net_ok(grad_critic)) return PR_EINVAL;
  static_assert(PR_STATIC_SCRATCH_BYTES == (size_t)24 << 20, "header and library disagree on the scratch size");
  if (ppo_static_scratch_bytes() != PR_STATIC_SCRATCH_BYTES ||
      !ppo_static_covers(cfg->batch, cfg->hidden, cfg->n_stocks, 1 + cfg->n_stocks * (2 + cfg->n_ind)))
    return PR_ETOOBIG;
  POD_HIP(launch_ppo_grads_static(static_cast<hipStream_t>(hip_stream), *cfg, obs, act_raw, logp_old, adv, ret, rows,
                                  *actor, *critic, *grad_actor, *grad_critic, stats));
  return PR_OK;
}

int adam_update(void *hip_stream, int64_t n, float *theta, const float *grad, float *m, float *v, float lr, float beta1,
                float beta2, float eps, int32_t t) {
  if (n < 1 || !theta || !grad || !m || !v || t < 1) return PR_EINVAL;
  if (!(beta1 >= 0.0f) || !(beta1 < 1.0f) || !(beta2 >= 0.0f) || !(beta2 < 1.0f) || !(eps > 0.0f) || !isfinite(lr))
    return PR_EINVAL;
  POD_HIP(launch_adam(static_cast<hipStream_t>(hip_stream), n, theta, grad, m, v, lr, beta1, beta2, eps, t));
  return PR_OK;
}

int ppo_learner_step(void *hip_stream, const pr_ppo_config *cfg, const float *obs, const float *act_raw,
                     const float *logp_old, const float *adv, const float *ret, const int32_t *rows,
                     const pr_net_params *actor, const pr_net_params *critic, const pr_net_params *m_actor,
                     const pr_net_params *v_actor, const pr_net_params *m_critic, const pr_net_params *v_critic,
                     void *workspace, size_t workspace_bytes, float *stats) {
  const int rc = ppo_config_ok(cfg);
  if (rc != PR_OK) return rc;
  if (!net_ok(m_actor) || !net_ok(v_actor) || !net_ok(m_critic) || !net_ok(v_critic) || !net_ok(actor) ||
      !net_ok(critic) || !workspace)
    return PR_EINVAL;
  if (cfg->adam_step < 1 || !(cfg->beta1 >= 0.0f) || !(cfg->beta1 < 1.0f) || !(cfg->beta2 >= 0.0f) ||
      !(cfg->beta2 < 1.0f) || !(cfg->adam_eps > 0.0f) || !isfinite(cfg->lr))
    return PR_EINVAL;
  const size_t scratch = ppo_scratch(*cfg, true);
  if ((reinterpret_cast<uintptr_t>(workspace) & 255u) || workspace_bytes < scratch + grads_bytes(*cfg)) return PR_EINVAL;
  // gradients behind the scratch, tensor by tensor
  unsigned char *p = static_cast<unsigned char *>(workspace) + scratch;
  int64_t na[6], nc[6];
  net_sizes(*cfg, cfg->n_stocks, na);
  net_sizes(*cfg, 1, nc);
  float *ga[6], *gc[6];
  for (int i = 0; i < 6; ++i) {
    ga[i] = reinterpret_cast<float *>(p);
    p += align_up((size_t)na[i] * 4, 256);
  }
  for (int i = 0; i < 6; ++i) {
    gc[i] = reinterpret_cast<float *>(p);
    p += align_up((size_t)nc[i] * 4, 256);
  }
  const pr_net_params gpa = {ga[0], ga[1], ga[2], ga[3], ga[4], ga[5]}, gpc = {gc[0], gc[1], gc[2], gc[3], gc[4], gc[5]};
  if (!obs || !act_raw || !logp_old || !adv || !ret) return PR_EINVAL;
  const PpoAdam adam = {{m_actor, m_critic}, {v_actor, v_critic}};
  POD_HIP(launch_ppo(static_cast<hipStream_t>(hip_stream), *cfg, obs, act_raw, logp_old, adv, ret, rows, *actor, *critic,
                     gpa, gpc, &adam, workspace, stats));
  return PR_OK;
}

int rollout_leaderboard(pr_handle *h, double *score_mean, double *score_var, int32_t *rank) {
  if (!h || !score_mean || !score_var || !rank) return PR_EINVAL;
  POD_HIP(launch_leaderboard(h->stream, h->cfg.n_envs, h->cfg.n_agents, h->st, nullptr, score_mean, score_var, rank));
  return PR_OK;
}

int rollout_calibrate(void *hip_stream, int32_t kind, int64_t n, const int32_t *params, void *buf_a, void *buf_b) {
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  if (!buf_a || !buf_b || n < 1) return PR_EINVAL;
  if (kind == PR_CAL_COPY || kind == PR_CAL_READ) {
    if (n % 16 != 0 || (reinterpret_cast<uintptr_t>(buf_a) & 15u) || (kind == PR_CAL_COPY && (reinterpret_cast<uintptr_t>(buf_b) & 15u)))
      return PR_EINVAL;
    const int blocks = 256 * 16;  // sixteen 256-thread workgroups per compute unit, grid-stride over the buffer
    POD_HIP(kind == PR_CAL_COPY ? launch_calib_copy(st, buf_a, buf_b, n, blocks) : launch_calib_read(st, buf_a, buf_b, n, blocks));
    return PR_OK;
  }
  if (kind != PR_CAL_PROBE || !params || n > 65535) return PR_EINVAL;
  bool any = false;
  for (int w = 0; w < 8; ++w) {
    if (params[w] < 0 || params[w] > 4) return PR_EINVAL;
    any = any || params[w] != 0;
  }
  if (!any || params[8] < 0 || params[9] < 0 || params[8] > (1 << 24) || params[9] > (1 << 24)) return PR_EINVAL;
  if (params[10] != 0 && params[10] != 2 && params[10] != 4 && params[10] != 6 && params[10] != 8) return PR_EINVAL;
  if (reinterpret_cast<uintptr_t>(buf_a) & 7u) return PR_EINVAL;
  POD_HIP(launch_calib_probe(st, params, params[8], params[9], params[10], params[11] != 0, (int)n,
                             static_cast<int64_t *>(buf_a), static_cast<float *>(buf_b)));
  return PR_OK;
}

int rollout_destroy(pr_handle *h) {
  if (!h) return PR_EINVAL;
  pthread_mutex_destroy(&h->enqueue);
  delete h;
  return PR_OK;
}

const char *rollout_strerror(int code) {
  switch (code) {
    case PR_OK: return "ok";
    case PR_EINVAL: return "invalid argument";
    case PR_ENOMEM: return "workspace too small or out of host memory";
    case PR_EHIP: return "HIP call failed";
    case PR_EUNSUPPORTED: return "shape or schedule not covered by the kernels";
    case PR_ETOOBIG: return "request needs more than the fixed scratch of this no-allocation entry point";
    default: return "unknown status";
  }
}

int rollout_last_hip_error(void) { return g_last_hip; }

}  // extern "C"
