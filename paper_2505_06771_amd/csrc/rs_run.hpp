// rs_run.hpp -- the persistent multi-step kernel over a work list of
// environments with mixed robot counts (used by env_run, env_reset_mixed, the
// autotuner and the serving loop).
#pragma once

#include "rs_internal.hpp"

namespace rs {

// Device view of one launch of the persistent kernel. Every per-env array is
// indexed by the env index e that the work list names.
struct RunArgs {
  SimConst<float> C;
  int E;           // rows of reward_out/done_out
  int steps;       // step budget of this launch
  int num_tiles;           // tiles of the launch (an upper bound when num_tiles_dev is set)
  const int32_t *num_tiles_dev;  // device tile count written by an earlier kernel (may be NULL)
  uint32_t env_base;
  uint32_t t0;
  const int4 *tiles;       // {G, first item, count, unused}
  const int32_t *items;    // env indices, tile after tile
  const int32_t *offset;   // [E] first robot of env e
  const int32_t *nrob;     // [E] robots of env e
  const uint32_t *env_ids; // [E] stream id of env e (NULL: env_base + e)
  const int64_t *t_start;  // [E] stream time of the env's first step (NULL: t0)
  int64_t *t_after;        // [E] written: t_start + steps run (may be NULL)
  const int32_t *steps_per_env;  // [E] step budget (NULL: steps)
  int32_t *steps_left_after;     // [E] written: budget - steps run (may be NULL)
  uint8_t *reset_mask;     // [E] reset (and clear) flagged envs first (may be NULL)
  const uint8_t *reset_only;  // [E] reset flagged envs, flags left as they are (may be NULL)
  int reset_all;           // reset every env first
  float *x, *y, *th, *gx, *gy;
  int32_t *step, *episode;
  float *reward_out;       // [steps][E] (may be NULL)
  uint8_t *done_out;       // [steps][E] (may be NULL)
  float *reward_sum;       // [E] accumulated (may be NULL)
  float *obs_final;        // (may be NULL)
  const int64_t *obs_off;  // [E] offsets into obs_final
  int32_t *qp_stats;       // [E][kQPStats] accumulated (may be NULL)
  unsigned long long *qp_fail;  // the context's failure counters
  int32_t qp_iters[17];
};

// Launch the persistent kernel: one wavefront per tile.
hipError_t launch_run(const RunArgs &A, int block_threads, hipStream_t st);

// Build tiles/items for the envs `envs` (indices) with robot counts `nrob_of`
// (indexed by env index), grouping by lanes-per-env from `sched`, on a device
// of `simds` SIMDs.
void build_tiles(const std::vector<int32_t> &envs, const std::vector<int32_t> &nrob_of,
                 const rs_schedule &sched, int simds, std::vector<int32_t> &tiles,
                 std::vector<int32_t> &items);

int lanes_for(const rs_schedule &sched, int n);

// Envs per wavefront tile for each robot count: the schedule's where it sets
// one (epw[n] > 0), else 64 / lanes, and less while that leaves SIMDs idle. A
// wavefront runs the solver stages that any of its envs needs, so fewer envs
// make its steps shorter. The largest teams, whose steps are the longest, come
// first: each takes the fewest envs per wavefront that keep the launch within
// one wavefront per SIMD, and in 16-lane groups within two, the most a SIMD
// holds: their solves stall more than they issue. Measured per step: 1024 envs
// of 8 in 128 wavefronts 2.20 us, in 1024 1.80 us; 3000 of 6 2.34 us in 750,
// 2.42 us in 1500; 2000 of 16 6.25 us in 1000, 6.02 us in 2000; 4096 of 12
// 4.56 us in 1024, 4.37 us in 2048 and 7.2 us in 4096; the mixed batch of 8192
// (2 to 12 robots) with its 12-robot envs four to a wavefront (898 in all)
// 3.91 us, three (966) 3.59 us, one (1512) 3.37 us.
template <typename Count>
__host__ __device__ inline void spread_envs(const Count *total, const int32_t *lanes, int simds,
                                            int32_t *epw) {
  bool automatic[RS_MAX_ROBOTS + 1];
  int tiles = 0;
  for (int n = 2; n <= RS_MAX_ROBOTS; ++n) {
    automatic[n] = epw[n] <= 0;
    if (automatic[n]) epw[n] = 64 / lanes[n];
    tiles += (int)((total[n] + epw[n] - 1) / epw[n]);
  }
  for (int n = RS_MAX_ROBOTS; n >= 2; --n) {
    if (!automatic[n] || total[n] == 0) continue;
    const int others = tiles - (int)((total[n] + epw[n] - 1) / epw[n]);
    const int room = (lanes[n] > 8 ? 2 * simds : simds) - others;
    if (room <= 0) continue;
    const int e = (int)((total[n] + room - 1) / room);
    if (e < epw[n]) {
      epw[n] = e;
      tiles = others + (int)((total[n] + e - 1) / e);
    }
  }
}
// The schedule's envs per wavefront for robot count n, 0 where it leaves them
// to spread_envs (bit n of envs_per_wave[0]: the value there is what
// spread_envs gave for the batch that the autotuner ran).
inline int scheduled_envs_per_wave(const rs_schedule &sched, int n) {
  if (((uint32_t)sched.envs_per_wave[0] >> n) & 1u) return 0;
  const int c = sched.envs_per_wave[n];
  return (c >= 1 && c <= 64 / lanes_for(sched, n)) ? c : 0;
}

}  // namespace rs
