// Kernels around the SAC chains of chains_sac.h (one launch per chain; the critic chain and
// the weight-gradient tiles are the TD3 ones).
#include <algorithm>
#include "chains_sac.h"

namespace pop {

// 64 rows: the nine scratch blocks leave no room for the slabs of the target and actor products
using SacRows64 = Rows32<2, false>;

// PER_CU: workgroups that share a CU (registers to match): two of the narrow 16-row chains, for tuning beyond 16 agents
template <class G, int PER_CU = 1>
__global__ __launch_bounds__(G::kThr, PER_CU * G::kThr / kThreads) void k_sac_target(PopDev d, uint32_t t) {
  warm_args<sizeof(PopDev) + 16>();
  extern __shared__ float lds[];
  int agent, chunk;
  POP_BLOCK_TIME(kTraceTarget, 0);
  if (decode_block(blockIdx.x, d.P, d.B / G::R, agent, chunk)) sac_target_chain<G>(d, t, agent, chunk, lds);
  POP_BLOCK_TIME(kTraceTarget, 1);
}

template <class G>
__global__ __launch_bounds__(G::kThr, G::kThr / kThreads) void k_sac_actor(PopDev d, uint32_t t) {
  warm_args<sizeof(PopDev) + 16>();
  extern __shared__ float lds[];
  int agent, chunk;
  POP_BLOCK_TIME(kTraceActor, 0);
  if (decode_block(blockIdx.x, d.P, d.B / G::R, agent, chunk)) sac_actor_chain<G>(d, t, agent, chunk, lds);
  POP_BLOCK_TIME(kTraceActor, 1);
}

// Target and critic chains in one launch, as for TD3 (k_chain.hip): the critics' forward pass runs beside
// the target workgroups and only the loss waits for the targets of its own rows.
template <class GT, class GC>
__global__ __launch_bounds__(kThreads, 1) void k_sac_target_critic(PopDev d, uint32_t t, int target_blocks) {
  warm_args<sizeof(PopDev) + 16>();
  extern __shared__ float lds[];
  int unit, chunk;
  POP_BLOCK_TIME(kTraceTargetCritic, 0);
  if ((int)blockIdx.x < target_blocks) {
    if (decode_block(blockIdx.x, d.P, d.B / GT::R, unit, chunk)) sac_target_chain<GT>(d, t, unit, chunk, lds);
  } else if (decode_block(blockIdx.x - target_blocks, 2 * d.P, d.B / GC::R, unit, chunk)) {
    critic_chain<GC, true, false>(d, t, unit, chunk, lds);
  }
  POP_BLOCK_TIME(kTraceTargetCritic, 1);
}

// The same for a few agents and for wide inputs (k_target_critic_few, k_few.hip).  SPLIT: a workgroup per target critic.
template <class GT, class GC, bool SPLIT>
__global__ __launch_bounds__(GT::kThr, GT::kThr / kThreads) void k_sac_target_critic_few(PopDev d, uint32_t t, int target_blocks) {
  static_assert(GT::kThr == GC::kThr, "one workgroup size");
  warm_args<sizeof(PopDev) + 16>();
  extern __shared__ float lds[];
  int unit, sub;
  POP_BLOCK_TIME(kTraceTargetCritic, 0);
  if ((int)blockIdx.x < target_blocks) {
    if (decode_block(blockIdx.x, d.P, (SPLIT ? 2 : 1) * (d.B / GT::R), unit, sub))
      sac_target_chain<GT, SPLIT>(d, t, unit, SPLIT ? sub >> 1 : sub, lds, sub & 1);
  } else if (decode_block(blockIdx.x - target_blocks, 2 * d.P, d.B / GC::R, unit, sub)) {
    critic_chain<GC, true, false, false, SPLIT, SPLIT>(d, t, unit, sub, lds);
  }
  POP_BLOCK_TIME(kTraceTargetCritic, 1);
}

hipError_t setup_sac_kernels() {
  hipError_t e;
  const int most = 160 * 1024;
#define POP_SET_LDS(...)                                                                                   \
  if ((e = hipFuncSetAttribute((const void*)__VA_ARGS__, hipFuncAttributeMaxDynamicSharedMemorySize, most)) != hipSuccess) return e
  POP_SET_LDS(k_sac_target<Rows16, 2>);
  POP_SET_LDS(k_sac_target<SacRows64>);
  POP_SET_LDS(k_sac_target<Rows16Deep>);
  POP_SET_LDS(k_sac_target<Rows32x8>);
  POP_SET_LDS(k_sac_target<Rows32Wide>);
  POP_SET_LDS(k_sac_actor<Rows16>);
  POP_SET_LDS(k_sac_actor<SacRows64>);
  POP_SET_LDS(k_sac_actor<Rows16Deep>);
  POP_SET_LDS(k_sac_actor<Rows32x8>);
  POP_SET_LDS(k_sac_actor<Rows32Wide>);
  POP_SET_LDS(k_sac_target_critic<Rows16, Rows32<2>>);
  POP_SET_LDS(k_sac_target_critic<Rows16, Rows32<1>>);
  POP_SET_LDS(k_sac_target_critic<Rows32<1>, Rows32<1>>);
  POP_SET_LDS(k_sac_target_critic_few<Rows16, Rows32<1>, true>);
  POP_SET_LDS(k_sac_target_critic_few<Rows16Deep, Rows32Deep<2, false>, true>);
  POP_SET_LDS(k_sac_target_critic_few<Rows16Deep, Rows32Deep<2, false>, false>);
  POP_SET_LDS(k_sac_target_critic_few<Rows32Wide, Rows32Wide, false>);
#undef POP_SET_LDS
  return hipSuccess;
}

size_t sac_lds_bytes(const PopDev& d) {
  auto chain = [&](int rows, int vec, bool back) {
    return rows == 16 ? chain_bytes<Rows16>(d.D, vec, back ? Rows16::kStage : Rows16::kStageForward, kSacScratch)
           : rows == 32 ? chain_bytes<Rows32<1>>(d.D, vec, Rows32<1>::kStage, kSacScratch)
                        : chain_bytes<SacRows64>(d.D, vec, SacRows64::kStage, kSacScratch);
  };
  size_t m = chain(d.rows_t, vec_sac_target(d), false);
  m = std::max(m, chain(d.rows_a, vec_sac_actor(d), true));
  m = std::max(m, d.rows_c == 32 ? chain_bytes<Rows32<1>>(d.D, vec_critic(d)) : chain_bytes<Rows32<2>>(d.D, vec_critic(d)));
  return std::max(m, act_lds_bytes(d));
}

hipError_t launch_sac_target(const PopDev& d, uint32_t t, hipStream_t s) {
  const dim3 grid(xcd_grid(d.P, d.B / d.rows_t)), block(kThreads);
  const int vec = vec_sac_target(d);
  if (d.D > kMaxIn) {                                // wide inputs: 16 rows, pipelined first layers
    if (d.rows_t == 16) k_sac_target<Rows16Deep><<<grid, block, chain_bytes<Rows16>(d.D, vec, Rows16::kStageForward, kSacScratch), s>>>(d, t);
    else if (d.rows_t == 32) k_sac_target<Rows32Wide><<<grid, dim3(Rows32x8::kThr), chain_bytes<Rows32<1>>(d.D, vec, Rows32<1>::kStage, kSacScratch), s>>>(d, t);
    else return hipErrorInvalidValue;
  } else if (d.rows_t == 16) k_sac_target<Rows16, 2><<<grid, block, chain_bytes<Rows16>(d.D, vec, Rows16::kStageForward, kSacScratch), s>>>(d, t);
  else if (d.rows_t == 32) k_sac_target<Rows32x8><<<grid, dim3(Rows32x8::kThr), chain_bytes<Rows32<1>>(d.D, vec, Rows32<1>::kStage, kSacScratch), s>>>(d, t);
  else k_sac_target<SacRows64><<<grid, block, chain_bytes<SacRows64>(d.D, vec, SacRows64::kStage, kSacScratch), s>>>(d, t);
  return hipGetLastError();
}

static hipError_t launch_sac_target_critic_few(const PopDev& d, uint32_t t, hipStream_t s) {
  const bool split = (d.spread & kSpreadTargets) != 0, wide = d.D > kMaxIn;
  if (d.rows_c != 32 || d.rows_c1 != 32 || (d.rows_t != 16 && (d.rows_t != 32 || split || !wide)) || (!wide && !split)) return hipErrorInvalidValue;
  const int nt = (split ? 2 : 1) * xcd_grid(d.P, d.B / d.rows_t), vec = vec_sac_target(d);
  const dim3 grid(nt + xcd_grid(2 * d.P, d.B / 32));
  if (d.rows_t == 32) {
    const size_t bytes = std::max(chain_bytes<Rows32<1>>(d.D, vec, Rows32<1>::kStage, kSacScratch), CriticMap<Rows32Wide>(d.D).bytes());
    k_sac_target_critic_few<Rows32Wide, Rows32Wide, false><<<grid, dim3(Rows32Wide::kThr), bytes, s>>>(d, t, nt);
    return hipGetLastError();
  }
  const size_t bytes = std::max(chain_bytes<Rows16>(d.D, vec, Rows16::kStageForward, kSacScratch),
                                wide ? CriticMap<Rows32Deep<2, false>>(d.D).bytes() : chain_bytes<Rows32<1>>(d.D, vec_critic(d)));
  auto* kernel = !wide ? k_sac_target_critic_few<Rows16, Rows32<1>, true>
                 : split ? k_sac_target_critic_few<Rows16Deep, Rows32Deep<2, false>, true> : k_sac_target_critic_few<Rows16Deep, Rows32Deep<2, false>, false>;
  kernel<<<grid, dim3(kThreads), bytes, s>>>(d, t, nt);
  return hipGetLastError();
}
hipError_t launch_sac_target_critic(const PopDev& d, uint32_t t, hipStream_t s) {
  if (d.spread || d.D > kMaxIn) return launch_sac_target_critic_few(d, t, s);
  const int nt = xcd_grid(d.P, d.B / d.rows_t), nc = xcd_grid(2 * d.P, d.B / d.rows_c);
  const dim3 grid(nt + nc), block(kThreads);
  const int vec = vec_sac_target(d);                 // larger than the critic chain's
  if (d.rows_t == 16 && d.rows_c == 64) {
    const size_t a = chain_bytes<Rows16>(d.D, vec, Rows16::kStageForward, kSacScratch), b = chain_bytes<Rows32<2>>(d.D, vec_critic(d));
    k_sac_target_critic<Rows16, Rows32<2>><<<grid, block, a > b ? a : b, s>>>(d, t, nt);
  } else if (d.rows_t == 16 && d.rows_c == 32) {
    const size_t a = chain_bytes<Rows16>(d.D, vec, Rows16::kStageForward, kSacScratch), b = chain_bytes<Rows32<1>>(d.D, vec_critic(d));
    k_sac_target_critic<Rows16, Rows32<1>><<<grid, block, a > b ? a : b, s>>>(d, t, nt);
  } else if (d.rows_t == 32 && d.rows_c == 32) {
    const size_t a = chain_bytes<Rows32<1>>(d.D, vec, Rows32<1>::kStage, kSacScratch), b = chain_bytes<Rows32<1>>(d.D, vec_critic(d));
    k_sac_target_critic<Rows32<1>, Rows32<1>><<<grid, block, a > b ? a : b, s>>>(d, t, nt);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_sac_actor(const PopDev& d, uint32_t t, hipStream_t s) {
  const dim3 grid(xcd_grid(d.P, d.B / d.rows_a)), block(kThreads);
  const int vec = vec_sac_actor(d);
  if (d.D > kMaxIn) {
    if (d.rows_a == 16) k_sac_actor<Rows16Deep><<<grid, block, chain_bytes<Rows16>(d.D, vec, Rows16::kStage, kSacScratch), s>>>(d, t);
    else if (d.rows_a == 32) k_sac_actor<Rows32Wide><<<grid, dim3(Rows32x8::kThr), chain_bytes<Rows32<1>>(d.D, vec, Rows32<1>::kStage, kSacScratch), s>>>(d, t);
    else return hipErrorInvalidValue;
  } else if (d.rows_a == 16) k_sac_actor<Rows16><<<grid, block, chain_bytes<Rows16>(d.D, vec, Rows16::kStage, kSacScratch), s>>>(d, t);
  else if (d.rows_a == 32) k_sac_actor<Rows32x8><<<grid, dim3(Rows32x8::kThr), chain_bytes<Rows32<1>>(d.D, vec, Rows32<1>::kStage, kSacScratch), s>>>(d, t);
  else k_sac_actor<SacRows64><<<grid, block, chain_bytes<SacRows64>(d.D, vec, SacRows64::kStage, kSacScratch), s>>>(d, t);
  return hipGetLastError();
}

}  // namespace pop
