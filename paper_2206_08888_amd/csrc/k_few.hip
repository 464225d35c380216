// The fused target / critic launch of a few TD3 agents and of wide inputs or actions.
#include <algorithm>
#include "chains.h"

namespace pop {

// Target and critic chains of one step in a single launch (as k_target_critic, k_chain.hip) for the few agents whose target (16 rows) and critic
// (32 rows) workgroups leave CUs idle, and for wide inputs or actions.  A step of so few agents is a chain of single-workgroup latencies, so the idle CUs take work out of
// it: SPLIT runs the two target critics in workgroups of their own (each repeats the target actor), and `ahead_blocks`
// workgroups run the actor's own forward pass.  Same sums, same bits.  Blocks: targets | forward passes | critics.  The 32-row chains of
// wide inputs or actions (eight wavefronts) have neither of the two.
template <class GT, class GC, int AS, bool SPLIT>
__global__ __launch_bounds__(GT::kThr, GT::kThr / kThreads) void k_target_critic_few(PopDev d, uint32_t t, int target_blocks, int ahead_blocks) {
  warm_args<sizeof(PopDev) + 16>();
  static_assert(GT::kThr == GC::kThr, "one workgroup size");
  extern __shared__ float lds[];
  int unit, sub, b = (int)blockIdx.x;
  POP_BLOCK_TIME(kTraceTargetCritic, 0);
  if (b < target_blocks) {
    if (decode_block(b, d.P, (SPLIT ? 2 : 1) * (d.B / GT::R), unit, sub))
      target_chain<GT, AS, SPLIT>(d, t, unit, SPLIT ? sub >> 1 : sub, lds, sub & 1);
  } else if ((b -= target_blocks) < ahead_blocks) {
    if constexpr (GT::R == 16)
      if (decode_block(b, d.P, d.B / GT::R, unit, sub)) actor_forward<GT, AS>(d, t, unit, sub, lds);
  } else if (decode_block(b - ahead_blocks, 2 * d.P, d.B / GC::R, unit, sub)) {
    critic_chain<GC, true, false, false, SPLIT>(d, t, unit, sub, lds);
  }
  POP_BLOCK_TIME(kTraceTargetCritic, 1);
}

hipError_t setup_few_kernels() {
  hipError_t e;
  const int most = 160 * 1024;
#define POP_SET_LDS(...)                                                                                   \
  if ((e = hipFuncSetAttribute((const void*)__VA_ARGS__, hipFuncAttributeMaxDynamicSharedMemorySize, most)) != hipSuccess) return e
  POP_SET_LDS(k_target_critic_few<Rows16, Rows32<1>, kMaxAct, true>);
  POP_SET_LDS(k_target_critic_few<Rows16Deep, Rows32Deep<2, false>, kMaxAct, true>);
  POP_SET_LDS(k_target_critic_few<Rows16Deep, Rows32Deep<2, false>, kMaxAct, false>);
  POP_SET_LDS(k_target_critic_few<Rows16Deep, Rows32Deep<2, false>, kSacMaxAct, true>);
  POP_SET_LDS(k_target_critic_few<Rows16Deep, Rows32Deep<2, false>, kSacMaxAct, false>);
  POP_SET_LDS(k_target_critic_few<Rows16Deep, Rows32<1>, kSacMaxAct, true>);
  POP_SET_LDS(k_target_critic_few<Rows16Deep, Rows32<1>, kSacMaxAct, false>);
  POP_SET_LDS(k_target_critic_few<Rows32Wide, Rows32Wide, kMaxAct, false>);
  POP_SET_LDS(k_target_critic_few<Rows32Wide, Rows32Wide, kSacMaxAct, false>);
  POP_SET_LDS(k_target_critic_few<Rows32Wide, Rows32x8, kSacMaxAct, false>);
#undef POP_SET_LDS
  return hipSuccess;
}

// wide inputs or actions, 32-row chains on eight wavefronts
static hipError_t launch_target_critic_wide(const PopDev& d, uint32_t t, hipStream_t s) {
  const int nt = xcd_grid(d.P, d.B / 32);
  const dim3 grid(nt + xcd_grid(2 * d.P, d.B / 32)), block(Rows32Wide::kThr);
  const int regions = d.A > kMaxAct ? kWideScratch : 3;
  const size_t bytes = std::max(chain_bytes<Rows32<1>>(d.D, vec_target(d), Rows32<1>::kStage, regions),
                                d.D > kMaxIn ? CriticMap<Rows32Wide>(d.D).bytes() : chain_bytes<Rows32<1>>(d.D, vec_critic(d)));
  auto* kernel = d.D <= kMaxIn   ? k_target_critic_few<Rows32Wide, Rows32x8, kSacMaxAct, false>      // wide actions alone: a critic's input is narrow
                 : d.A > kMaxAct ? k_target_critic_few<Rows32Wide, Rows32Wide, kSacMaxAct, false>
                                 : k_target_critic_few<Rows32Wide, Rows32Wide, kMaxAct, false>;
  kernel<<<grid, block, bytes, s>>>(d, t, nt, 0);
  return hipGetLastError();
}
hipError_t launch_target_critic_few(const PopDev& d, uint32_t t, hipStream_t s) {
  if (d.rows_t == 32 && d.rows_c == 32 && d.rows_c1 == 32 && !d.spread && !d.w2_plain) return launch_target_critic_wide(d, t, s);
  if (d.rows_t != 16 || d.rows_c != 32 || d.rows_c1 != 32 || d.w2_plain) return hipErrorInvalidValue;
  const bool split = (d.spread & kSpreadTargets) != 0;
  const int chunks = xcd_grid(d.P, d.B / 16), nt = split ? 2 * chunks : chunks, na = d.spread & kSpreadActor ? chunks : 0;
  const dim3 grid(nt + na + xcd_grid(2 * d.P, d.B / 32)), block(kThreads);
  const int vec = std::max(std::max(vec_target(d), vec_actor(d)), vec_critic(d));
  if (d.D <= kMaxIn && d.A <= kMaxAct) {
    if (!split) return hipErrorInvalidValue;         // k_target_critic has it
    const size_t bytes = std::max(chain_bytes<Rows16>(d.D, vec, Rows16::kStageForward), chain_bytes<Rows32<1>>(d.D, vec));
    k_target_critic_few<Rows16, Rows32<1>, kMaxAct, true><<<grid, block, bytes, s>>>(d, t, nt, na);
    return hipGetLastError();
  }
  const size_t bytes = std::max(chain_bytes<Rows16>(d.D, vec, Rows16::kStageForward, d.A > kMaxAct ? kWideScratch : 3),
                                d.D > kMaxIn ? CriticMap<Rows32Deep<2, false>>(d.D).bytes() : chain_bytes<Rows32<1>>(d.D, vec));
  auto* kernel = d.D <= kMaxIn  ? (split ? k_target_critic_few<Rows16Deep, Rows32<1>, kSacMaxAct, true>     // wide actions alone: a critic's input is narrow
                                         : k_target_critic_few<Rows16Deep, Rows32<1>, kSacMaxAct, false>)
                 : d.A > kMaxAct ? (split ? k_target_critic_few<Rows16Deep, Rows32Deep<2, false>, kSacMaxAct, true>
                                        : k_target_critic_few<Rows16Deep, Rows32Deep<2, false>, kSacMaxAct, false>)
                               : (split ? k_target_critic_few<Rows16Deep, Rows32Deep<2, false>, kMaxAct, true>
                                        : k_target_critic_few<Rows16Deep, Rows32Deep<2, false>, kMaxAct, false>);
  kernel<<<grid, block, bytes, s>>>(d, t, nt, na);
  return hipGetLastError();
}
}  // namespace pop
