// Internal declarations shared by the HIP translation units of libpodrollout.
// Host-side launchers only; every kernel lives in the .hip file that defines
// its launcher.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "podrollout.h"

namespace pod {

// Kernels that use more than the default 64 KiB of dynamic LDS need the limit raised once per device (the
// attribute belongs to that device's copy of the code object).  One bit per device ordinal and kernel; safe to
// call from several host threads (a second call on a device is harmless).
constexpr int kMaxLdsBytes = 160 * 1024;
template <auto Kern>
inline hipError_t allow_full_lds() {
  static std::atomic<uint64_t> done{0};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = 1ull << (dev & 63);
  if (dev < 64 && (done.load(std::memory_order_acquire) & bit)) return hipSuccess;
  e = hipFuncSetAttribute(reinterpret_cast<const void *>(Kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                          kMaxLdsBytes);
  if (e != hipSuccess) return e;
  if (dev < 64) done.fetch_or(bit, std::memory_order_release);
  return hipSuccess;
}

// ---------------------------------------------------------------- env state
// Structure-of-arrays env state in the workspace; a tile of consecutive envs
// is one contiguous segment of every array.
struct EnvState {
  float *cash;       // [N]
  int32_t *tau;      // [N]
  int32_t *h;        // [N][D]
  double *ep_ret;    // [N]
  double *ep_sum;    // [N]
  double *ep_sqsum;  // [N]
  int32_t *ep_cnt;   // [N]
  const int32_t *start;  // [N] table row every episode of the env begins at (0 unless a replay table is set)
};

struct EnvDims {
  int32_t N, D, K, S, H, M;
  float cash0, hmax, one_minus_c, one_plus_c, sigma, rho;
  float logp_const;  // -D * (ln sigma + 0.5 ln 2 pi)
  float s_cash, s_price, s_hold, s_ind;
};

// Market rows of a step by the cursor rule (whole numbers only).
struct RowInfo {
  int32_t row_now;   // market row the trades execute at
  int32_t row_val;   // market row the portfolio is valued at (cursor + 1)
  int32_t row_obs;   // market row of the next observation (of the env's start row after a reset)
  int32_t done;
};

__device__ inline RowInfo rows_of(const EnvDims &d, int32_t tau, int32_t start, int32_t n) {
  const int32_t m = d.M == 1 ? 0 : n;
  RowInfo r;
  r.row_now = tau * d.M + m;
  r.row_val = (tau + 1) * d.M + m;
  r.done = (tau + 1 - start == d.H);
  r.row_obs = r.done ? start * d.M + m : r.row_val;
  return r;
}

// Observations in bf16 as the layer-per-launch actor reads them: [N][pitch], columns in the order of its rotated first
// layer [indicators | cash | prices | holdings | zeros].
struct ObsShadow {
  uint16_t *p;
  int32_t pitch, cols;  // elements; columns up to `cols` are read
};

struct StepIO {
  const float *mu;     // [N, D] policy mean of this step
  const float *noise;  // [N, D]
  float *obs_next;     // [N, S] observation after the step
  float *act_raw;      // [N, D]
  float *reward;       // [N]
  uint8_t *done;       // [N]
  float *logp;         // [N] or null
  int32_t *shares;     // [N, D] or null
  ObsShadow shadow;    // the next observation for the actor, or null
  bool ind_done;       // the next observation's indicators are there already (IndicatorMove)
};

// Indicators of the observation after a step, which need nothing the step computes: launch_layers moves them beside the
// policy's second or third layer (the first one reads the shadow they go to) where that leaves compute units idle, and
// says so.
struct IndicatorMove {
  EnvDims d;
  EnvState s;
  const float *ind;
  float *obs_next;
  ObsShadow shadow;
  bool moved;
};

hipError_t launch_observe(hipStream_t st, const EnvDims &d, const EnvState &s, const float *price, const float *ind,
                          float *obs, const ObsShadow &shadow);
hipError_t launch_env_step(hipStream_t st, const EnvDims &d, const EnvState &s, const float *price, const float *ind,
                           const StepIO &io);
hipError_t launch_state_reset(hipStream_t st, const EnvDims &d, const EnvState &s);
hipError_t launch_check_starts(hipStream_t st, int32_t N, int32_t H, int32_t rows, const int32_t *start, int32_t *bad);
hipError_t launch_state_copy(hipStream_t st, const EnvDims &d, const EnvState &s, const pr_state &user, bool to_user);
hipError_t launch_leaderboard(hipStream_t st, int32_t N, int32_t P, const EnvState &s, double *scratch_mean,
                              double *score_mean, double *score_var, int32_t *rank);

// ---------------------------------------------------------------------- GAE
// obs_scale: host pointer to the four observation scales.
hipError_t launch_trading_metrics(hipStream_t st, int32_t T, int32_t N, int32_t D, int32_t S, const float *obs,
                                  const uint8_t *done, const float *obs_scale, double periods, double rf,
                                  double *metrics, int32_t *length);
hipError_t launch_population_refill(hipStream_t st, int32_t P, int64_t count, const int32_t *rank, int32_t keep,
                                    float sigma, const float *noise, float *params);
size_t ppo_scratch_bytes(int B, int Hd, int D, int S, bool adam);
// Gradients into ga / gc (whose tensors also hold intermediate sums), and with `adam` the update of both networks.
struct PpoAdam {
  const pr_net_params *m[2], *v[2];  // actor, critic
};
hipError_t launch_ppo(hipStream_t st, const pr_ppo_config &c, const float *obs, const float *act, const float *logp_old,
                      const float *adv, const float *ret, const int32_t *rows, const pr_net_params &actor,
                      const pr_net_params &critic, const pr_net_params &ga, const pr_net_params &gc,
                      const PpoAdam *adam, void *scratch, float *stats);
// The same with the scratch in a fixed device array of ppo_static_scratch_bytes() (no workspace, no allocation);
// hipErrorInvalidValue for the shapes it is not for.
size_t ppo_static_scratch_bytes();
bool ppo_static_covers(int B, int Hd, int D, int S);
hipError_t launch_ppo_grads_static(hipStream_t st, const pr_ppo_config &c, const float *obs, const float *act,
                                   const float *logp_old, const float *adv, const float *ret, const int32_t *rows,
                                   const pr_net_params &actor, const pr_net_params &critic, const pr_net_params &ga,
                                   const pr_net_params &gc, float *stats);
hipError_t launch_adam(hipStream_t st, int64_t n, float *theta, const float *g, float *m, float *v, float lr, float b1,
                       float b2, float eps, int32_t t);
hipError_t launch_gae(hipStream_t st, int32_t T, int32_t N, const float *reward, const float *value,
                      const uint8_t *done, float gamma, float lambda, float *adv, float *ret);

// -------------------------------------------------------------- calibration
hipError_t launch_calib_copy(hipStream_t st, const void *src, void *dst, int64_t bytes, int blocks);
hipError_t launch_calib_read(hipStream_t st, const void *src, void *sink, int64_t bytes, int blocks);
hipError_t launch_calib_probe(hipStream_t st, const int32_t role_of_wave[8], int32_t iters_matrix,
                              int32_t iters_vector, int32_t acts_per_group, int32_t lds_reads, int blocks,
                              int64_t *ticks, float *sink);

// ---------------------------------------------------------------------- MLP
// Packed network of one agent set.  Weight blocks are stored in the register
// layout of the matrix-core instruction: block (kb, ct) holds, for the 64 lanes
// of a wavefront, the 16 bytes lane l feeds as operand for output features
// [32 ct, 32 ct + 32) and inputs [16 kb, 16 kb + 16); for fp32, three such blocks with the parts of the split values.
// Blocks are ordered k-major: [kb][ct][lane].
struct PackedNet {
  const void *W[3];       // packed weights per layer, agent-major
  const float *b[3];      // biases padded to a multiple of 32, agent-major
  int64_t w_stride[3];    // bytes between agents
  int32_t b_stride[3];    // floats between agents
  int32_t in_dim[3], out_dim[3];  // logical sizes
  int32_t nkb[3], nct[3];         // k-blocks and column tiles per layer
  int32_t bf16;                   // operand type
  int32_t out_tanh;               // tanh on the last layer
  void *split_h[2];               // scratch for the layer-per-launch path: two buffers of split_rows rows of hidden
                                  // activations (fp32 [hidden] or bf16 [layers_pitch(hidden)]), or null
  ObsShadow split_x;              // and, for bf16 networks, of its input
  int64_t split_rows;
};
// Rows the scratch of the layer-per-launch paths holds: all envs where a step's rows can take one of them (fewer 64-row
// tiles than half the compute units), and always enough for a policy asked about a few; 0 for networks too narrow for them.
int64_t split_scratch_rows(int64_t n_envs, int hidden);

size_t packed_weight_bytes(int in_dim, int out_dim, int bf16);
int padded_out(int out_dim);
// Inputs `at` .. `at` + count - 1 of a packed layer are rows `row` .. of its weights.
struct PackRun {
  int32_t at, row, count;
};
// One layer to pack, in nkb k-blocks: its rows in up to three runs, zeros elsewhere.
struct PackJob {
  const float *W, *b;  // [P, in_dim, out_dim], [P, out_dim]
  void *Wp;
  float *bp;
  int32_t in_dim, out_dim, nkb;
  PackRun run[3];
};
// three layers of two networks, and the actor's first layer in the rollout's order or both first layers in their parts
constexpr int kMaxPackJobs = 10;
hipError_t launch_pack_layers(hipStream_t st, const PackJob *jobs, int n, int P, int bf16);
// rows of X [rows, ldx] -> Y [rows, out_dim[2]]; row r uses agent ((r % N) / envs_per_agent).
hipError_t launch_mlp(hipStream_t st, const PackedNet &net, int64_t rows, const float *X, int64_t ldx, float *Y,
                      int32_t N, int32_t envs_per_agent);
// The fp32 value head with 256 hidden units over many dense rows, on `cus` compute units: with several agents whole steps
// of N rows, whose envs per agent are a multiple of 32.
bool value_rows_covers(int64_t rows, int32_t N, int32_t envs_per_agent);
hipError_t launch_value_rows(hipStream_t st, const PackedNet &net, int64_t rows, const float *X, float *Y, int32_t N,
                             int32_t envs_per_agent, int cus);
bool mlp_supported(int S, int Hd, int O, int bf16);
int compute_units();  // of the device the library was first used on
// The bf16 layer-per-launch path: x holds the rows (columns up to x.cols zero-padded) in the order layer 1 was packed for.
bool layers_supported(int64_t rows, int hidden, int bf16);
// the hidden layers of two networks side by side over N rows are a workgroup or less per compute unit
bool layers_room_beside(int32_t N, int32_t envs_per_agent, int hidden);
int32_t layers_pitch(int cols);
hipError_t launch_layers(hipStream_t st, const PackedNet &net, int64_t rows, const ObsShadow &x, float *Y, int32_t N,
                         int32_t envs_per_agent, IndicatorMove *move = nullptr, const PackedNet *beside = nullptr);
// `beside`: the hidden layers of a second network of the same shape on the same rows, in the same launches, into its split_h;
// launch_hidden: those of one network alone.  launch_value_dot: a value head's output layer on rows of such activations.
hipError_t launch_hidden(hipStream_t st, const PackedNet &net, int64_t rows, const ObsShadow &x, int32_t N, int32_t envs_per_agent);
hipError_t launch_value_dot(hipStream_t st, const PackedNet &net, int64_t rows, const void *h, float *Y, int32_t N, int32_t envs_per_agent);
// Few rows of either operand type: a launch per layer that splits the inputs over a workgroup's wavefronts.  `converted`:
// the alternative has its rows in bf16 already.
bool few_rows(int64_t rows, int S, int hidden, int bf16, bool converted);
hipError_t launch_few_rows(hipStream_t st, const PackedNet &net, int64_t rows, const float *X, int64_t ldx, float *Y,
                           int32_t N, int32_t envs_per_agent);
// Few rows of networks whose weights pass through one compute unit quickly: all layers in one launch that keeps nothing.
bool query_supported(int64_t rows, int S, int hidden, int outputs, int bf16, int32_t N, int32_t envs_per_agent);
// and where a launch per layer, if there is scratch for it, is the faster one all the same
bool query_outweighed(int64_t rows, int S, int hidden, int bf16, bool several);
hipError_t launch_query(hipStream_t st, const PackedNet &net, int64_t rows, const float *X, int64_t ldx, float *Y, int32_t N,
                        int32_t envs_per_agent);
// The output layer alone, on bf16 activations [rows][pitch].
hipError_t launch_rows_output(hipStream_t st, const PackedNet &net, int64_t rows, const void *h, int64_t pitch, float *Y,
                              int32_t N, int32_t envs_per_agent);
hipError_t launch_rows_to_bf16(hipStream_t st, int64_t rows, const float *X, int64_t ldx, int S, const ObsShadow &out);

// ------------------------------------------------------- persistent rollout
// One launch for T steps: each workgroup keeps 64 envs on its compute unit (actor forward, sampling, trading
// step, observation assembly).  mu_forced != null replaces the actor by caller-supplied means.
bool fused_supported(const pr_config &c);
size_t fused_lds_bytes(const pr_config &c, bool with_actor);
hipError_t launch_rollout_fused(hipStream_t st, const pr_config &c, const EnvDims &d, const EnvState &s,
                                const float *price, const float *ind, const PackedNet &actor, int32_t envs_per_agent,
                                int32_t T, const float *noise, const float *mu_forced, const pr_buffers &out);

// The same with the actor for fp32 networks.
size_t fused_f32_lds_bytes(const pr_config &c);
hipError_t launch_rollout_fused_f32(hipStream_t st, const EnvDims &d, const EnvState &s, const float *price, const float *ind,
                                    const PackedNet &actor, int32_t envs_per_agent, int32_t T, const float *noise,
                                    const pr_buffers &out);

// The stepwise schedule of small networks: all T steps in one launch, state and network on the compute units.
bool small_supported(const pr_config &c);
hipError_t launch_rollout_small(hipStream_t st, const EnvDims &d, const EnvState &s, const float *price, const float *ind,
                                const PackedNet &actor, int32_t envs_per_agent, int32_t T, const float *noise,
                                const pr_buffers &out);

// And the value head over the observations of such a rollout, whole steps of N rows, on `cus` compute units.
// (the rows it is the fastest kernel for)
bool value_small_covers(const PackedNet &critic, int64_t rows);
hipError_t launch_value_small(hipStream_t st, const PackedNet &critic, int64_t rows, const float *X, int32_t S, float *Y, int32_t N,
                              int32_t envs_per_agent, int cus);

// Stepwise rollouts of bf16 networks over one shared market table (pod_table.hip): the market part of layer 1 is formed per
// table row into P (or per env and step, where those are fewer or the table is longer than P), everything else in one launch.
bool table_supported(const pr_config &c);
int table_market_blocks(int D, int K);
int table_portfolio_blocks(int D);
int64_t table_rows_kept(int64_t n_envs, int64_t horizon);
size_t table_scratch_bytes(int64_t n_envs, int64_t horizon);
struct TableMarket {
  const float *price, *ind;
  int32_t rows;
};
struct TableNet {
  const void *Wm, *Wp;    // layer 1: inputs [indicators | prices], and [holdings | zeros | cash]
  const void *W[3];       // the layers behind it
  const float *b[3];
};
// tau0: [N], receives the cursors the call starts at.
hipError_t launch_rollout_table(hipStream_t st, const EnvDims &d, const EnvState &s, const TableMarket &m, const TableNet &actor,
                                float *P, int32_t *tau0, int32_t T, const float *noise, const pr_buffers &out, int cus);
// The value head over the observations of such a rollout, where they are many for the table's rows.
bool value_table_covers(int64_t rows, int S, int32_t n_envs, int32_t horizon, int32_t table_rows);
hipError_t launch_value_table(hipStream_t st, const EnvDims &d, const EnvState &s, const TableMarket &m, const TableNet &critic,
                              float *P, const int32_t *tau0, int64_t rows, const float *obs, float *Y, int cus);

}  // namespace pod
