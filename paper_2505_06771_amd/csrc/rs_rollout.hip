// rs_rollout.hip -- C-ABI entry point of the fused policy rollout, and its
// kernels with full wavefronts (64 / G envs each).
#include "rs_rollout.hpp"

#include <algorithm>

namespace rs {

#ifdef RS_PHASE_TIMERS
// Per-wavefront phase cycles of the last rollout launch (diagnostic builds).
__device__ unsigned long long rs_phase_cycles_dev[kTimedWaves][kPhases];
#endif

// Kernel for N = 2..14 robots.
template <bool PP, bool ST> static const void *full_kernel(int N) {
  const void *k = nullptr;
  static_for<2, 15>([&](auto nc) {
    constexpr int n = decltype(nc)::value;
    constexpr int g = n <= 2 ? 2 : (n <= 4 ? 4 : (n <= 8 ? 8 : 16));
    if (N == n) k = reinterpret_cast<const void *>(&k_rollout<g, n, PP, ST, false>);
  });
  return k;
}
static const void *rollout_kernel(const RolloutArgs &A) {
  const bool pp = A.C.scenario == RS_SCN_PREDATOR_PREY, st = A.qp_stats != nullptr;
  if (A.epw < 64 / pow2_group(A.N)) return rollout_split_kernel(A.N, pp);
  if (pp) return st ? full_kernel<true, true>(A.N) : full_kernel<true, false>(A.N);
  return st ? full_kernel<false, true>(A.N) : full_kernel<false, false>(A.N);
}

static bool launch_rollout(const RolloutArgs &A, dim3 grid, hipStream_t st) {
  RolloutArgs copy = A;
  void *kargs[] = {&copy};
  return hipLaunchKernel(rollout_kernel(A), grid, dim3(kRollBlock), kargs, 0, st) == hipSuccess;
}

}  // namespace rs

using namespace rs;

extern "C" rs_status rollout(rs_ctx *ctx, const rs_params *p, const rs_batch *b,
                             const rs_policy *policy, int32_t horizon, int64_t t_global0,
                             float *obs, uint8_t *actions, float *reward, uint8_t *done,
                             int32_t *qp_stats, void *stream) {
  RS_CHECK_ARG(ctx != nullptr, "ctx is NULL");
  rs_status s = check_params(p);
  if (s != RS_OK) return s;
  RS_CHECK_ARG(b != nullptr && policy != nullptr, "batch/policy is NULL");
  RS_CHECK_ARG(p->dtype == RS_F32, "rollout runs in FP32 (dtype must be RS_F32)");
  RS_CHECK_ARG(action_driven(p->controller), "rollout samples actions: discrete, waypoint or pose controller");
  RS_CHECK_ARG(b->num_envs >= 1, "num_envs must be >= 1");
  RS_CHECK_ARG((int64_t)b->num_envs * b->robots < (int64_t)1 << 31, "num_envs * robots must be < 2^31");
  RS_CHECK_ARG(b->robots >= 2 && 2 * b->robots + 4 <= 32,
               "rollout needs 2 <= robots and 2*robots+4 <= 32 (got %d)", b->robots);
  RS_CHECK_ARG(horizon >= 1, "horizon must be >= 1");
  RS_CHECK_ARG(policy->in_dim == 2 * b->robots + 4, "policy in_dim %d != 2N+4", policy->in_dim);
  RS_CHECK_ARG(policy->w1 && policy->w2 && policy->w3 && policy->b1 && policy->b2 && policy->b3,
               "policy pointer is NULL");
  RS_CHECK_ARG(actions && reward && done, "actions/reward/done outputs are required");
  RS_CHECK_ARG(b->x && b->y && b->theta && b->goal_x && b->goal_y && b->step && b->episode,
               "state pointer is NULL");
  RS_CHECK_ARG(((uintptr_t)obs & 15) == 0, "obs must be 16-byte aligned");
  RolloutArgs A;
  std::memset(&A, 0, sizeof(A));
  A.C = make_const<float>(*p);
  A.E = b->num_envs;
  A.N = b->robots;
  A.D = 2 * b->robots + 4;
  A.H = horizon;
  A.env_base = (uint32_t)b->env_id_base;
  A.t0 = (uint32_t)t_global0;
  A.x = (float *)b->x; A.y = (float *)b->y; A.th = (float *)b->theta;
  A.gx = (float *)b->goal_x; A.gy = (float *)b->goal_y;
  A.step = b->step; A.episode = b->episode;
  A.w1 = (const __bf16 *)policy->w1; A.w2 = (const __bf16 *)policy->w2;
  A.w3 = (const __bf16 *)policy->w3;
  A.b1 = policy->b1; A.b2 = policy->b2; A.b3 = policy->b3;
  A.obs = obs; A.actions = actions; A.reward = reward; A.done = done;
  A.qp_stats = qp_stats;
  A.qp_fail = ctx->qp_fail;
  const int G = pow2_group(A.N);
  // Envs per wavefront. A step is one long dependency chain, and a wavefront
  // runs the solver stages that any of its envs needs, so while SIMDs are idle
  // fewer envs per wavefront make a shorter step: 4.5 -> 2.3 us at 96 x 6 (12
  // -> 96 wavefronts), 3.9 -> 3.0 us at 2048 x 8 (256 -> 1024). Above 32 lanes
  // the tiles of the split kernel run one after the other, and with two
  // wavefronts per SIMD full ones win. A step at 4096 x 8 with 512 (full), 1024
  // and 2048 wavefronts: 3.9, 3.4 and 5.2 us; 6000 x 8 with 750 and 1500: 3.9 and
  // 5.8; 4096 x 3 with 256, 512, 1024 and 2048: 3.2, 2.4, 2.1 and 3.7; 2048 x 12
  // with 512, 1024 and 2048: 6.3, 5.2 and 7.7. Calls with qp_stats take full
  // wavefronts (no counting kernels with split ones), so a small batch's step is
  // up to twice as long in them.
  const int full = 64 / G, simds = 4 * ctx->num_cus;
  A.epw = full;
  if (!qp_stats)
    for (int n = 1; n * G <= 32 && A.epw == full; n *= 2)
      if ((A.E + n - 1) / n <= simds) A.epw = n;
  const int waves = (A.E + A.epw - 1) / A.epw;
  const dim3 grid((waves + kRollWaves - 1) / kRollWaves);
  hipStream_t st = (hipStream_t)stream;
#ifdef RS_PHASE_TIMERS
  RS_CHECK_HIP(hipGetSymbolAddress((void **)&A.phase, HIP_SYMBOL(rs_phase_cycles_dev)));
#endif

  // Replay a captured graph of this launch shape; when only scalar arguments
  // (e.g. the stream time) differ, patch the kernel node of the instantiated
  // graph instead of capturing again.
  RolloutArgs shape = A;
  shape.t0 = 0;
  GraphKey key;
  key.words.resize((sizeof(A) + sizeof(uintptr_t) - 1) / sizeof(uintptr_t) + 1, 0);
  std::memcpy(key.words.data(), &shape, sizeof(shape));
  key.words.back() = grid.x;
  auto it = ctx->graphs.find(key);
  if (it == ctx->graphs.end()) {
    if (ctx->graphs.size() >= 32) {
      for (auto &kv : ctx->graphs) {
        (void)hipGraphExecDestroy(kv.second.exec);
        (void)hipGraphDestroy(kv.second.graph);
      }
      ctx->graphs.clear();
    }
    if (!ctx->capture_stream)
      RS_CHECK_HIP(hipStreamCreateWithFlags(&ctx->capture_stream, hipStreamNonBlocking));
    CachedGraph cg;
    RS_CHECK_HIP(hipStreamBeginCapture(ctx->capture_stream, hipStreamCaptureModeThreadLocal));
    const bool ok = launch_rollout(A, grid, ctx->capture_stream);
    hipError_t ce = hipStreamEndCapture(ctx->capture_stream, &cg.graph);
    if (!ok || ce != hipSuccess) {
      set_error("rollout capture failed: %s", hipGetErrorString(ce));
      return RS_ERR_DEVICE;
    }
    size_t nnodes = 1;
    hipError_t ne = hipGraphGetNodes(cg.graph, &cg.node, &nnodes);
    hipError_t ie = hipGraphInstantiate(&cg.exec, cg.graph, nullptr, nullptr, 0);
    if (ne != hipSuccess || nnodes != 1 || ie != hipSuccess) {
      set_error("rollout graph instantiate failed: %s", hipGetErrorString(ie));
      if (cg.graph) (void)hipGraphDestroy(cg.graph);
      return RS_ERR_DEVICE;
    }
    cg.args.assign(reinterpret_cast<const char *>(&A), reinterpret_cast<const char *>(&A) + sizeof(A));
    it = ctx->graphs.emplace(key, cg).first;
  } else if (std::memcmp(it->second.args.data(), &A, sizeof(A)) != 0) {
    RolloutArgs copy = A;
    void *kargs[] = {&copy};
    hipKernelNodeParams kp;
    std::memset(&kp, 0, sizeof(kp));
    kp.func = const_cast<void *>(rollout_kernel(A));
    kp.gridDim = grid;
    kp.blockDim = dim3(kRollBlock);
    kp.sharedMemBytes = 0;
    kp.kernelParams = kargs;
    kp.extra = nullptr;
    RS_CHECK_HIP(hipGraphExecKernelNodeSetParams(it->second.exec, it->second.node, &kp));
    std::memcpy(it->second.args.data(), &A, sizeof(A));
  }
  RS_CHECK_HIP(hipGraphLaunch(it->second.exec, st));
  return RS_OK;
}

extern "C" rs_status rs_phase_cycles(rs_ctx *ctx, int64_t *out, int32_t waves) {
  RS_CHECK_ARG(ctx != nullptr && out != nullptr && waves >= 1, "ctx/out/waves invalid");
#ifdef RS_PHASE_TIMERS
  RS_CHECK_ARG(waves <= kTimedWaves, "at most %d wavefronts are recorded", kTimedWaves);
  RS_CHECK_HIP(hipSetDevice(ctx->device));
  RS_CHECK_HIP(hipDeviceSynchronize());
  RS_CHECK_HIP(hipMemcpyFromSymbol(out, HIP_SYMBOL(rs_phase_cycles_dev),
                                   (size_t)waves * kPhases * sizeof(int64_t), 0,
                                   hipMemcpyDeviceToHost));
  return RS_OK;
#else
  set_error("phase timers are compiled out (build with RS_PHASE_TIMERS)");
  return RS_ERR_UNSUPPORTED;
#endif
}
