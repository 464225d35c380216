// Host-side launch wrappers implemented in the kernel source files.
#pragma once
#include <hip/hip_runtime.h>
#include "pop_dev.h"

namespace pop {

// parameter initialisation: Glorot-uniform weights of the three online networks
// of every agent, copied into the targets; limits are computed by the host.
struct InitLimits { float actor[3], critic[3]; };
hipError_t launch_init(const PopDev& d, const InitLimits& lim, hipStream_t s);

// replay ring: write n rows per agent starting at cursor (agent < 0: all agents,
// sources carry a leading population axis), then advance cursor and count.
hipError_t launch_insert(const PopDev& d, int agent, int64_t n, const float* obs, const float* act,
                         const float* rew, const float* done, const float* next_obs, hipStream_t s);

// one update step
hipError_t launch_sample_gather(const PopDev& d, uint32_t t, hipStream_t s);
hipError_t launch_target(const PopDev& d, uint32_t t, hipStream_t s);
hipError_t launch_critic(const PopDev& d, uint32_t t, hipStream_t s);
hipError_t launch_target_critic(const PopDev& d, uint32_t t, hipStream_t s);   // both of the above in one launch
hipError_t launch_target_critic_few(const PopDev& d, uint32_t t, hipStream_t s);   // the same for a few agents and wide shapes (k_few.hip)
hipError_t setup_few_kernels();
// What a fused target / critic launch of 16-row target and 32-row critic chains has CUs left for (kSpread*); `forward`: the actor's forward pass is wanted there.
inline int spread_of(const PopDev& d, bool forward) {
  if (d.rows_t != 16 || d.rows_c != 32 || d.rows_c1 != 32 || d.rows_a != 16 || d.actor_ahead) return 0;
  const int64_t b16 = (int64_t)d.P * (d.B / 16), chains = b16 + 2 * (int64_t)d.P * (d.B / 32);
  return (chains + b16 <= kCUs ? kSpreadTargets : 0) | (forward && chains + 2 * b16 <= kCUs ? kSpreadActor : 0);
}
bool wide_critics_alone(const PopDev& d);   // wide inputs: a critic workgroup's LDS leaves no room for a second one on its CU
hipError_t launch_actor(const PopDev& d, uint32_t t, hipStream_t s);
// prefetch_next != 0: extra workgroups also gather the replay rows of step t + 1
hipError_t launch_wgrad_adam(const PopDev& d, uint32_t t, int actor_phase, int prefetch_next, hipStream_t s);

// shared critics: partial gradient sums per agent group, then Adam on the one critic pair (k_wgrad_shared.hip)
hipError_t launch_wgrad_shared(const PopDev& d, uint32_t t, int prefetch_next, hipStream_t s);

// SAC: target chain (online actor, soft clipped double-Q target) and actor chain (k_sac.hip); the critic chain
// and the weight-gradient launches are shared with TD3
hipError_t launch_sac_target(const PopDev& d, uint32_t t, hipStream_t s);
hipError_t launch_sac_actor(const PopDev& d, uint32_t t, hipStream_t s);
hipError_t launch_sac_target_critic(const PopDev& d, uint32_t t, hipStream_t s);   // target + critic chains in one launch
hipError_t setup_sac_kernels();
size_t act_lds_bytes(const PopDev& d);   // dynamic LDS of the acting kernel
size_t td3_lds_bytes(const PopDev& d);   // largest dynamic LDS request of the TD3 step's and the acting kernels
size_t sac_lds_bytes(const PopDev& d);   // the same for the SAC step

// the step as one launch (k_step.hip); with_chains = 0: without the target and critic chains (launched
// before); with_actor: some agent has its delayed actor step at t; launch_seq: 0, 1, 2, ... over the
// launches of this kernel on this population (alternates the two sets of hand-over counters)
hipError_t launch_step(const PopDev& d, uint32_t t, uint32_t launch_seq, int with_chains, int with_actor,
                       int prefetch_next, hipStream_t s);
hipError_t setup_step_kernel();
int wgrad_role_count(const PopDev& d, int actor_phase);

// acting: obs[P][n][O] -> act[P][n][A] through the online actors; a noise scale above zero adds exploration noise drawn at counter
// `step`, rows numbered from row_base.  The scales: sigma (device, [P]), or where that is nullptr those of `args` (up to
// kStaticMaxP agents; they travel as a kernel argument); both nullptr: no noise.  `whole`: rows of the caller's request, of
// which this launch may be a piece: it decides which kernel and which form of its head runs, so that a row comes out the same in one piece and in several.
constexpr int kStaticMaxP = 256;
struct SigmaArgs { float s[kStaticMaxP]; };
constexpr SigmaArgs kNoNoise{};
hipError_t launch_act(const PopDev& d, const float* obs, int n, float* act, const float* sigma, const SigmaArgs* args, uint32_t step,
                      uint32_t row_base, int whole, hipStream_t s);
// Grid of k_act: x = `chunks` blocks of 32 rows per agent, y = pieces of that many.  A dimension of a grid holds fewer than 2^32 threads and what
// is beyond is cut off without an error, so a request of more than 2^24 - 1 workgroups of 256 (537 million rows of all agents) takes several pieces.
struct ActGrid { int chunks, pieces; };
inline ActGrid act_grid(int P, int n) {
  const int64_t all = ((int64_t)n + 31) / 32, most = ((1 << 24) - 1) / P;
  const int64_t chunks = all < most ? all : most;
  return {(int)chunks, (int)((all + chunks - 1) / chunks)};
}
hipError_t launch_act_rows(const PopDev& d, const float* obs, int n, float* act, const float* sigma, const SigmaArgs* args, uint32_t step,
                           uint32_t row_base, int whole, hipStream_t s);
hipError_t setup_act_kernels();

// one-time per-process kernel attribute setup (large dynamic LDS)
hipError_t setup_kernels();

}  // namespace pop
