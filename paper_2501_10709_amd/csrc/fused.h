// The fused rollout: ensemble MLP (bfloat16 MFMA), noise, trading, reward and next state for
// every step of a rollout in one launch (fused_rollout.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <string>
#include <type_traits>

#include "device_common.h"
#include "mlp_device.h"

namespace fm {

// Days of noise that the fused rollout's scratch holds, and steps per launch of the batched form.
constexpr int kFusedChunk = 64;
// Scratch floats of the split-layer schedules for N environments and D stocks: the noise
// [kFusedChunk][N][D] and market table [kFusedChunk][8][512] (any supported K, H).
inline size_t fused_eps_floats(size_t N, size_t D) { return static_cast<size_t>(kFusedChunk) * N * D; }
inline size_t fused_table_floats() { return static_cast<size_t>(kFusedChunk) * 8 * 512; }

// Arguments of a fused launch over a span of steps.
struct FusedArgs {
  int t0, n_steps;
  float sigma;
  uint64_t key;
  int64_t env_offset;
  float* obs_traj;
  float* act_traj;
  double* rew_traj;
  int* qty_traj;
  const float* eps;  // streamed and resident schedules: the launch's noise [n_steps][N][D] (may be act_traj)
  const float* mt;   // streamed and resident schedules: the launch's layer-1 market shares [n_steps][K][H]
  int tile_envs = 0; // streamed and resident schedules: environments per workgroup
};

// Environments per workgroup of the resident schedule (one compute unit each).
constexpr int kResRows = 8;

// Rows (environments) per workgroup of the fused kernel: 16 * row_tiles.
struct FusedTuning {
  int row_tiles = 0;  // streamed: 0 chooses from the problem size
  int schedule = 0;   // 0: resident when the shape allows and N fills at most one workgroup per
                      // compute unit, else wide when the shape allows, else streamed when it
                      // allows that; 1: streamed when the shape allows; 2: always the generic
                      // schedule; 3: resident whenever the shape allows
  int tile_envs = 0;  // resident / wide / streamed: environments per workgroup, 0: fill the compute units
};

// True when the streamed MLP schedule handles this ensemble and environment.
bool fused_streamed_shape(const EnvConst& C, const EnsDev& E);
// True when the resident schedule (weights held on chip) handles them.
bool fused_resident_shape(const EnvConst& C, const EnsDev& E);

// The market table mt[c][k][j] of days t .. t+n-1 (actor k's layer-1 share of day t+c's market
// entries, bias included), for ensembles that split their first layer.
hipError_t launch_market_table(const EnvConst& C, const EnsDev& E, int t, int n, float* mt, hipStream_t stream);
// The noise eps[c][n][d] of days t .. t+n-1.
hipError_t launch_noise(const EnvConst& C, int t, int n, uint64_t key, int64_t env_offset, float* eps, hipStream_t stream);

// Runs F's steps as launches of as many days as their inputs have room for: launch(Fc) per span of
// days, after its market table and noise.  The table's scratch holds kFusedChunk days of the largest
// ensemble, which is more days of a smaller one; the noise goes into the rows that the actions are
// stored to, if they are (a kernel reads an environment's noise of a day before it writes its actions
// there, and reads no other's), else through kFusedChunk days of scratch.  So a rollout of 252 days
// that stores its actions is one launch of each kind and not four (each sets up the weights anew).
template <class Launch>
hipError_t launch_spans(const EnvConst& C, const EnsDev& E, const FusedArgs& F, float* eps_chunk, float* mt_chunk,
                        hipStream_t stream, Launch launch) {
  const size_t N = C.N, D = C.D, S = C.S;
  const int table_days = static_cast<int>(fused_table_floats() / (static_cast<size_t>(E.K) * E.H));
  // Without noise too: the streamed kernel reads its rows (and leaves them unused) at any sigma.
  const bool scratch = !F.act_traj;
  const int days = scratch && kFusedChunk < table_days ? kFusedChunk : table_days;
  for (int i = 0; i < F.n_steps; i += days) {
    const int n = F.n_steps - i < days ? F.n_steps - i : days;
    FusedArgs Fc = F;
    Fc.t0 = F.t0 + i;
    Fc.n_steps = n;
    Fc.mt = mt_chunk;
    Fc.obs_traj = F.obs_traj ? F.obs_traj + i * N * S : nullptr;
    Fc.act_traj = F.act_traj ? F.act_traj + i * N * D : nullptr;
    Fc.rew_traj = F.rew_traj ? F.rew_traj + i * N : nullptr;
    Fc.qty_traj = F.qty_traj ? F.qty_traj + i * N * D : nullptr;
    float* eps = scratch ? eps_chunk : Fc.act_traj;
    Fc.eps = eps;
    hipError_t err = launch_market_table(C, E, Fc.t0, n, mt_chunk, stream);
    if (err == hipSuccess && F.sigma != 0.0f) err = launch_noise(C, Fc.t0, n, F.key, F.env_offset, eps, stream);
    if (err == hipSuccess) err = launch(Fc);
    if (err != hipSuccess) return err;
  }
  return hipSuccess;
}

// The resident schedule over F's steps (fused_resident.hip).
hipError_t launch_resident(const EnvConst& C, const EnvState& st, const EnsDev& E, FusedArgs F, float* eps_chunk,
                           float* mt_chunk, hipStream_t stream);

// One launch of the wide resident schedule (fused_wide.hip): the resident schedule's shapes, up to 32
// environments per workgroup.
hipError_t launch_wide_chunk(const EnvConst& C, const EnvState& st, const EnsDev& E, const FusedArgs& F,
                             hipStream_t stream);

// Returns hipSuccess and leaves *why empty on success; sets *why for unsupported shapes.
hipError_t launch_fused_rollout(const EnvConst& C, const EnvState& st, const EnsDev& E, int t0,
                                int n_steps, float sigma, uint64_t key, int64_t env_offset,
                                float* obs_traj, float* act_traj, double* rew_traj, int* qty_traj,
                                float* eps_chunk, float* mt_chunk, hipStream_t stream, std::string* why,
                                FusedTuning tune = FusedTuning());

// Batched persistent rollout of uneven groups (generic schedule, hidden size 256, K <= 8; the
// first layer split into per-environment rows and a per-day market table when the ensemble
// packs it so).
// rows: environments per work item (16 or 32).  A group descriptor is an opaque block of
// batched_group_desc_bytes() bytes, filled on the host and copied to the device.
size_t batched_lds_bytes(int rows, const EnvConst& C, const EnsDev& E);
size_t batched_group_desc_bytes();
// mt: the group's market-table slot ([kFusedChunk][K][H] floats, refilled before each chunk by
// launch_market_table) when the ensemble splits its first layer, else ignored.
void batched_group_desc(const EnvConst& C, const EnvState& st, const EnsDev& E, int t0, int n_steps, float sigma,
                        uint64_t key, int64_t env_offset, float* obs_traj, float* act_traj, double* rew_traj,
                        int* qty_traj, const float* mt, void* out);
// The batched kernels' dynamic LDS limit: raised to lds (<= batched_max_lds()) outside any
// stream capture.
size_t batched_max_lds();
hipError_t prepare_batched(size_t lds);
// actors: the most that a group has; items: int2 (group, tile) pairs; counter: one int of device scratch.
hipError_t launch_batched(int rows, int actors, int blocks, size_t lds, const void* groups, const int* items, int n_items,
                          int* counter, hipStream_t stream);

}  // namespace fm
