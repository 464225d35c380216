// Kernels around the layer chains of chains.h, one launch per chain:
//   k_target, k_critic, k_actor : the three chains of an update step
//   k_target_critic             : target and critic chains in one launch
//   k_act                       : obs -> actor (acting, no gradient)
#include <algorithm>
#include "chains.h"

namespace pop {

// PER_CU: wavefronts that share a SIMD (registers to match), i.e. workgroups per CU where they have four.
template <class G, int PER_CU = G::kPerSimd, int AS = kMaxAct>
__global__ __launch_bounds__(G::kThr, PER_CU) void k_target(PopDev d, uint32_t t) {
  warm_args<sizeof(PopDev) + 16>();
  extern __shared__ float lds[];
  int agent, chunk;
  POP_BLOCK_TIME(kTraceTarget, 0);
  if (decode_block(blockIdx.x, d.P, d.B / G::R, agent, chunk)) target_chain<G, AS>(d, t, agent, chunk, lds);
  POP_BLOCK_TIME(kTraceTarget, 1);
}

template <class G>
__global__ __launch_bounds__(G::kThr, G::kPerSimd) void k_critic(PopDev d, uint32_t t) {
  warm_args<sizeof(PopDev) + 16>();
  extern __shared__ float lds[];
  int net, chunk;
  POP_BLOCK_TIME(kTraceCritic, 0);
  if (decode_block(blockIdx.x, 2 * d.P, d.B / G::R, net, chunk)) critic_chain<G, false, false>(d, t, net, chunk, lds);
  POP_BLOCK_TIME(kTraceCritic, 1);
}

// Target and critic chains of one step in a single launch.  The critic's forward pass does
// not need the Bellman targets, so its workgroups run beside the target workgroups and
// only wait, before the loss, for the targets of their own rows.  Target workgroups have the
// lower block indices: workgroups are dispatched in index order, so whatever a critic
// workgroup waits for has already been dispatched and the wait always ends.
// GT, GC: tile geometries of the two chains.  AHEAD: critic_chain's.
template <class GT, class GC, bool AHEAD = false>
__global__ __launch_bounds__(GT::kThr, GT::kPerSimd < GC::kPerSimd ? GT::kPerSimd : GC::kPerSimd) void k_target_critic(PopDev d, uint32_t t, int target_blocks) {
  warm_args<sizeof(PopDev) + 16>();
  static_assert(GT::kThr == GC::kThr, "one workgroup size");
  extern __shared__ float lds[];
  int unit, chunk;
  POP_BLOCK_TIME(kTraceTargetCritic, 0);
  if ((int)blockIdx.x < target_blocks) {
    if (decode_block(blockIdx.x, d.P, d.B / GT::R, unit, chunk)) target_chain<GT>(d, t, unit, chunk, lds);
  } else if (decode_block(blockIdx.x - target_blocks, 2 * d.P, d.B / GC::R, unit, chunk)) {
    critic_chain<GC, true, false, AHEAD>(d, t, unit, chunk, lds);
  }
  POP_BLOCK_TIME(kTraceTargetCritic, 1);
}

// The same for populations whose 16-row target workgroups and 32-row critic workgroups do not all get a CU at
// once: a target workgroup goes on into critic 1 for its own 16 rows (its targets are its own, nothing waits),
// and only critic 2 has workgroups of its own.  GC: its geometry; the target workgroups read the hidden matrices in the same order.
//
// Its chains read more of the kernel's arguments than there are scalar registers.  Left to itself, the compiler requests all of them at the
// start and spills them as they arrive, up to three trips to memory one after the other; here the target chains' arguments are requested
// together, and the critic chains read theirs, through a pointer of their own, where they begin (10 agents: launch 40.0 -> 39.7 us, 73.7 ->
// 73.3 us/step).
__device__ inline const PopDev& late_args() {
  auto p = (const __attribute__((address_space(4))) PopDev*)__builtin_amdgcn_kernarg_segment_ptr();   // the first argument
  asm volatile("" : "+s"(p));
  return *(const PopDev*)p;
}
__device__ inline void request_together(const NetLayout& L) { asm volatile("" ::"s"(L.in), "s"(L.w1), "s"(L.b1), "s"(L.w2), "s"(L.b2), "s"(L.w3), "s"(L.b3)); }
__device__ inline void request_together(const PopDev& d) {
  asm volatile("" ::"s"(d.share), "s"(d.P), "s"(d.O), "s"(d.A), "s"(d.D), "s"(d.B), "s"(d.row), "s"(d.agent_sz), "s"(d.hp), "s"(d.batch));
}
template <class GC, bool AHEAD = false>
__global__ __launch_bounds__(kThreads, 1) void k_target_critic1(PopDev d, uint32_t t, int target_blocks) {
  extern __shared__ float lds[];
  int agent, chunk;
  asm volatile("" ::"s"(t), "s"(target_blocks), "s"(d.target));
  request_together(d);
  request_together(d.actor);
  request_together(d.critic);
  using GT = Rows16In<GC::kPlain>;
  POP_BLOCK_TIME(kTraceTargetCritic, 0);
  if ((int)blockIdx.x < target_blocks) {
    if (decode_block(blockIdx.x, d.P, d.B / 16, agent, chunk)) {
      target_chain<GT>(d, t, agent, chunk, lds);
      __syncthreads();                               // the chain is done with its LDS; a lane reads back the targets it wrote
      critic_chain<GT, false, false>(late_args(), t, 2 * agent, chunk, lds);
    }
  } else if (decode_block(blockIdx.x - target_blocks, d.P, d.B / GC::R, agent, chunk)) {
    critic_chain<GC, true, false, AHEAD>(late_args(), t, 2 * agent + 1, chunk, lds);
  }
  POP_BLOCK_TIME(kTraceTargetCritic, 1);
}

// PER_CU: wavefronts per SIMD the register budget is set for; AHEAD, AS: actor_chain's
template <class G, int PER_CU = G::kThr / kThreads, bool AHEAD = false, int AS = kMaxAct>
__global__ __launch_bounds__(G::kThr, PER_CU) void k_actor(PopDev d, uint32_t t) {
  if constexpr (G::kThr != kThreads || PER_CU == 1) warm_args<sizeof(PopDev) + 16>();       // (the other is short of registers: 2 more spilled)
  extern __shared__ float lds[];
  int agent, chunk;
  POP_BLOCK_TIME(kTraceActor, 0);
  if (decode_block(blockIdx.x, d.P, d.B / G::R, agent, chunk)) actor_chain<G, false, AHEAD, AS>(d, t, agent, chunk, lds, 0);
  POP_BLOCK_TIME(kTraceActor, 1);
}

// ---------------------------------------------------------------------------------------------
// Acting: act[agent][r] = pi_agent(obs[agent][r]).  A workgroup per agent and 32 rows, those of an agent on one XCD: numbered row block by row block
// they lay on all eight, and each L2 fetched every agent's weights (80 agents x 1000 rows 91.1 -> 84.8 us, 256 x 300 100.0 -> 85.9, 80 x 300 of 376
// inputs 159 -> 137; the head on all four wavefronts is part of it).
// Noise scale sigma[agent] > 0: Gaussian exploration noise, a = clip(pi + sigma[agent] eps, -1, 1) with eps =
// unit normal number (row_base + r) A + j of the agent's exploration stream at counter `step`
// (row_base: index of row 0 of this call within the caller's whole request).  Grid: act_grid.
// NOISE: whether the call has noise scales.  Read behind the head they cost one scalar trip; read with the weights, in one kernel for both, they stood
// in front of the LDS accesses, which are waited for with them.  us, read early / a kernel for each: with noise, 70 agents 125 rows of 269 inputs
// 46.96 / 46.34, 13 SAC agents 1409 rows 38.2 / 37.9; without, 3 SAC agents 777 rows 12.75 / 12.74 (read behind the head in one kernel for both: 12.88).
template <bool PLAIN, bool NOISE>
__global__ __launch_bounds__(kThreads) void k_act(PopDev d, const float* __restrict__ obs, int n,
                                                  float* __restrict__ act, const float* __restrict__ sigma, uint32_t step,
                                                  uint32_t row_base, int chunks, int share_head, SigmaArgs sigma_args) {
  warm_args<sizeof(PopDev) + 48>();
  constexpr int R = 32;
  extern __shared__ float lds[];
  constexpr int kHs = kMaxHead;                      // row stride of the head block
  const ActMap L(d.O);
  float* Xs = lds + L.input;
  float* buf = lds + L.buf;
  float* head = lds + L.head;
  float* v_ab3 = lds + L.bias;
  float* stage = Xs;                                 // the input tile is done with when the hidden layer starts
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  int agent, chunk;
  if (chunks == 1) { agent = blockIdx.x; chunk = 0; }                      // what decode_block makes of it, without its divisions
  else if (!decode_block(blockIdx.x, d.P, chunks, agent, chunk)) return;   // an agent's chunks share an XCD's L2 for its weights
  chunk += blockIdx.y * chunks;
  if (chunk > (n - 1) / R) return;                   // past the end of the last piece
  const int r0 = chunk * R;
  const int valid = n - r0 < R ? n - r0 : R;
  const float* an = net_ptr(d, d.theta, agent, 0);
  LayerPre<1, 2, PLAIN> pre;
  pre.load(an, d.actor, wave, lane);
  const float* rows = obs + ((size_t)agent * n + r0) * d.O;
  if (d.O <= kMaxIn) {                               // one trip to memory for all of the prologue
    SmallVec ab3;
    InputTile<R> xin;
    ab3.fetch(an + d.actor.b3, d.actor.out, tid);
    xin.fetch(L.xld, rows, d.O, 0, d.O, valid, tid);
    ab3.put(v_ab3, d.actor.out, tid);
    xin.put(Xs, L.xld, tid);
  } else {
    stage_vector(v_ab3, an + d.actor.b3, d.actor.out, tid);
    load_input_wide<R>(Xs, L.xld, rows, d.O, 0, d.O, valid, tid);
  }
  __syncthreads();
  first_layer<1, false>(Xs, L.xld, an, d.actor, pre, buf, nullptr, wave, lane);
  __syncthreads();
  hidden_layer<1, false, true>(buf, an, d.actor, pre, nullptr, wave, lane, NoTail(), stage);
  __syncthreads();
  // SAC: 2A outputs, the means come first
  if (share_head) head_mfma_split<R, false>(buf, an + d.actor.w3, d.actor.out, head, kHs, wave, lane, stage);
  else head_mfma<R>(buf, an + d.actor.w3, d.actor.out, head, kHs, wave, lane);
  const bool sac = d.algo == 1;
  float sg = 0.0f;
  uint32_t seed_lo = 0u, seed_hi = 0u;
  if constexpr (NOISE) {
    sg = sigma ? sigma[agent] : sigma_args.s[agent < kStaticMaxP ? agent : 0];
    seed_lo = d.hp[agent].seed_lo;
    seed_hi = d.hp[agent].seed_hi;
  }
  __syncthreads();
  for (int e = tid; e < valid * d.A; e += kThreads) {
    const int r = e / d.A, j = e - r * d.A;
    const float pre_act = head[r * kHs + j] + v_ab3[j];
    float a = tanhf(pre_act);
    if (NOISE && sg > 0.0f) {
      const uint32_t el = (row_base + (uint32_t)(r0 + r)) * (uint32_t)d.A + (uint32_t)j;
      const U4 blk = philox4x32_10(seed_lo, seed_hi, el >> 2, step, kStreamExplore, 0u);
      float n4[4];
      normals4(blk, n4);
      const float nz = (el & 2u) ? ((el & 1u) ? n4[3] : n4[2]) : ((el & 1u) ? n4[1] : n4[0]);
      if (sac) {                                     // a sample of the policy itself, its std scaled by sigma
        const float ls = fminf(fmaxf(head[r * kHs + d.A + j] + v_ab3[d.A + j], -20.0f), 2.0f);
        a = tanhf(pre_act + sg * expf(ls) * nz);
      } else {
        a = fminf(fmaxf(a + sg * nz, -1.0f), 1.0f);
      }
    }
    act[((size_t)agent * n + r0 + r) * d.A + j] = a;
  }
}

hipError_t setup_kernels() {
  hipError_t e;
  const int most = 160 * 1024;                        // whole LDS of a CU; the launches ask for what they need
#define POP_SET_LDS(...)                                                                                   \
  if ((e = hipFuncSetAttribute((const void*)__VA_ARGS__, hipFuncAttributeMaxDynamicSharedMemorySize, most)) != hipSuccess) return e
  POP_SET_LDS(k_target<Rows16Deep, 1, kSacMaxAct>);
  POP_SET_LDS(k_target<Rows32Deep<2>, 2, kSacMaxAct>);
  POP_SET_LDS(k_actor<Rows16Deep, 1, false, kSacMaxAct>);
  POP_SET_LDS(k_target<Rows16Deep>);
  POP_SET_LDS(k_target<Rows32Deep<2>, 2>);
  POP_SET_LDS(k_target<Rows32x8>);
  POP_SET_LDS(k_target<Rows32Wide>);
  POP_SET_LDS(k_target<Rows32Wide, 2, kSacMaxAct>);
  POP_SET_LDS(k_actor<Rows16Deep>);
  POP_SET_LDS(k_target<Rows16>);
  POP_SET_LDS(k_target<Rows32<1>>);
  POP_SET_LDS(k_target<Rows64>);
  POP_SET_LDS(k_critic<Rows32<1>>);
  POP_SET_LDS(k_critic<Rows32x8>);
  POP_SET_LDS(k_critic<Rows32Wide>);
  POP_SET_LDS(k_critic<Rows64>);
  POP_SET_LDS(k_critic<Rows32Deep<2, false>>);
  POP_SET_LDS(k_actor<Rows16>);
  POP_SET_LDS(k_actor<Rows32x8>);
  POP_SET_LDS(k_actor<Rows32Wide>);
  POP_SET_LDS(k_actor<Rows32Wide, 2, false, kSacMaxAct>);
  POP_SET_LDS(k_actor<Rows32<1>, 2>);
  POP_SET_LDS(k_actor<Rows32<2>>);
  POP_SET_LDS(k_target_critic<Rows16, Rows32<2>>);
  POP_SET_LDS(k_target_critic<Rows16, Rows32<1>>);
  POP_SET_LDS(k_target_critic1<Rows32<1>>);
  POP_SET_LDS(k_target_critic1<Rows32<2>>);
  POP_SET_LDS(k_target_critic1<Rows32<1>, true>);
  POP_SET_LDS(k_target_critic1<Rows32<1, true, 2, true>>);
  POP_SET_LDS(k_target_critic1<Rows32<2, true, 2, true>>);
  POP_SET_LDS(k_target_critic1<Rows32<1, true, 2, true>, true>);
  POP_SET_LDS(k_actor<Rows16In<true>>);
  POP_SET_LDS(k_actor<Rows16In<true>, 1, true>);
  POP_SET_LDS(k_target_critic<Rows16, Rows32<1>, true>);
  POP_SET_LDS(k_actor<Rows16Deep, 1, true>);
  POP_SET_LDS(k_actor<Rows16Deep, 1, true, kSacMaxAct>);
  POP_SET_LDS(k_actor<Rows16, 1, true>);
  POP_SET_LDS(k_target_critic<Rows32<1>, Rows32<1>>);
  POP_SET_LDS(k_target_critic<Rows64, Rows64>);
  POP_SET_LDS((k_act<false, false>));
  POP_SET_LDS((k_act<false, true>));
  POP_SET_LDS((k_act<true, false>));
  POP_SET_LDS((k_act<true, true>));
#undef POP_SET_LDS
  return hipSuccess;
}

// Rows per workgroup (pop_dev.h): (target, critic, actor) = (16, 32 or 64, 16) for small
// populations, else (32, 32, 32), from 104 agents on (64, 64, 64); shared critics from 56 on (64, 64, 32).
// LDS of the largest chain workgroup of a TD3 step at these shapes (the launches below ask for what each needs)
size_t td3_lds_bytes(const PopDev& d) {
  auto chain = [&](int rows, int vec, bool back, int regions) {
    return rows == 16 ? chain_bytes<Rows16>(d.D, vec, back ? Rows16::kStage : Rows16::kStageForward, regions)
           : rows == 32 ? chain_bytes<Rows32<1>>(d.D, vec, Rows32<1>::kStage, regions)
                        : chain_bytes<Rows32<2>>(d.D, vec, Rows32<2>::kStage, regions);
  };
  const int regions = d.A > kMaxAct ? kWideScratch : 3;
  size_t m = chain(d.rows_t, vec_target(d), false, regions);
  m = std::max(m, chain(d.rows_c, vec_critic(d), true, 3));
  m = std::max(m, chain(d.rows_a, vec_actor(d), true, regions));
  return std::max(m, act_lds_bytes(d));
}
size_t act_lds_bytes(const PopDev& d) { return ActMap(d.O).bytes(); }

hipError_t launch_target(const PopDev& d, uint32_t t, hipStream_t s) {
  const dim3 grid(xcd_grid(d.P, d.B / d.rows_t)), block(kThreads);
  const bool alone = (int)grid.x <= kCUs;            // a CU to each workgroup; the LDS may leave no other choice
  if (d.A > kMaxAct) {                               // wide actions: scratch rows of kSacMaxAct floats, first layers as for wide inputs
    const size_t b32 = chain_bytes<Rows32<1>>(d.D, vec_target(d), Rows32<1>::kStage, kWideScratch);
    if (d.rows_t == 16) k_target<Rows16Deep, 1, kSacMaxAct><<<grid, block, chain_bytes<Rows16>(d.D, vec_target(d), Rows16::kStageForward, kWideScratch), s>>>(d, t);
    else if (d.rows_t == 32 && (alone || 2 * b32 > (size_t)kLdsPerCU)) k_target<Rows32Wide, 2, kSacMaxAct><<<grid, dim3(Rows32x8::kThr), b32, s>>>(d, t);
    else if (d.rows_t == 32) k_target<Rows32Deep<2>, 2, kSacMaxAct><<<grid, block, b32, s>>>(d, t);
    else return hipErrorInvalidValue;
  } else if (d.D > kMaxIn) {                         // wide inputs: pipelined first layers, 16 or 32 rows
    const size_t b32 = chain_bytes<Rows32<1>>(d.D, vec_target(d));
    if (d.rows_t == 16) k_target<Rows16Deep><<<grid, block, chain_bytes<Rows16>(d.D, vec_target(d), Rows16::kStageForward), s>>>(d, t);
    else if (d.rows_t == 32 && (alone || 2 * b32 > (size_t)kLdsPerCU)) k_target<Rows32Wide><<<grid, dim3(Rows32x8::kThr), b32, s>>>(d, t);
    else if (d.rows_t == 32) k_target<Rows32Deep<2>, 2><<<grid, block, b32, s>>>(d, t);
    else return hipErrorInvalidValue;
  } else if (d.rows_t == 16) k_target<Rows16><<<grid, block, chain_bytes<Rows16>(d.D, vec_target(d), Rows16::kStageForward), s>>>(d, t);
  else if (d.rows_t == 32 && alone) k_target<Rows32x8><<<grid, dim3(Rows32x8::kThr), chain_bytes<Rows32<1>>(d.D, vec_target(d)), s>>>(d, t);
  else if (d.rows_t == 32) k_target<Rows32<1>><<<grid, block, chain_bytes<Rows32<1>>(d.D, vec_target(d)), s>>>(d, t);
  else k_target<Rows64><<<grid, dim3(Rows64::kThr), chain_bytes<Rows32<2>>(d.D, vec_target(d)), s>>>(d, t);
  return hipGetLastError();
}
bool wide_critics_alone(const PopDev& d) { return d.D > kMaxIn && 2 * CriticMap<Rows32Deep<2, false>>(d.D).bytes() > (size_t)kLdsPerCU; }
hipError_t launch_critic(const PopDev& d, uint32_t t, hipStream_t s) {
  const dim3 grid(xcd_grid(2 * d.P, d.B / d.rows_c)), block(kThreads);
  if (d.D > kMaxIn) {                                // wide inputs: 32 rows, pipelined first layer
    if (d.rows_c != 32) return hipErrorInvalidValue;
    const size_t over = CriticMap<Rows32Deep<2, false>>(d.D).bytes(), beside = CriticMap<Rows32Wide>(d.D).bytes();
    if (wide_critics_alone(d) || (int)grid.x <= kCUs)                // a CU to itself in any case
      k_critic<Rows32Wide><<<grid, dim3(Rows32Wide::kThr), beside, s>>>(d, t);
    else k_critic<Rows32Deep<2, false>><<<grid, block, over, s>>>(d, t);
  } else if (d.rows_c == 32 && (int)grid.x <= kCUs) k_critic<Rows32x8><<<grid, dim3(Rows32x8::kThr), chain_bytes<Rows32<1>>(d.D, vec_critic(d)), s>>>(d, t);
  else if (d.rows_c == 32) k_critic<Rows32<1>><<<grid, block, chain_bytes<Rows32<1>>(d.D, vec_critic(d)), s>>>(d, t);
  else k_critic<Rows64><<<grid, dim3(Rows64::kThr), chain_bytes<Rows32<2>>(d.D, vec_critic(d)), s>>>(d, t);
  return hipGetLastError();
}
hipError_t launch_target_critic(const PopDev& d, uint32_t t, hipStream_t s) {
  if (d.spread || d.D > kMaxIn || d.A > kMaxAct) return launch_target_critic_few(d, t, s);
  const int nt = xcd_grid(d.P, d.B / d.rows_t), nc = xcd_grid(2 * d.P, d.B / d.rows_c);
  const int vec = vec_target(d) > vec_critic(d) ? vec_target(d) : vec_critic(d);
  if (d.rows_c1 != d.rows_c) {                       // critic 1 inside the target workgroups
    if (d.rows_t != 16 || d.rows_c1 != 16 || (d.rows_c != 32 && d.rows_c != 64)) return hipErrorInvalidValue;
    // (the 16-row critic chain stages the weights of its transposed product in LDS)
    const size_t a = chain_bytes<Rows16>(d.D, vec), b = d.rows_c == 32 ? chain_bytes<Rows32<1>>(d.D, vec) : chain_bytes<Rows32<2>>(d.D, vec);
    const dim3 grid(nt + xcd_grid(d.P, d.B / d.rows_c)), block(kThreads);
    if (d.actor_ahead) {
      if (d.rows_c != 32) return hipErrorInvalidValue;
      const size_t c = Lds<1>(d.D).bytes(kAheadBase + ahead_floats<32>());
      if (d.w2_plain) k_target_critic1<Rows32<1, true, 2, true>, true><<<grid, block, a > c ? a : c, s>>>(d, t, nt);
      else k_target_critic1<Rows32<1>, true><<<grid, block, a > c ? a : c, s>>>(d, t, nt);
    } else if (d.rows_c == 32) {
      if (d.w2_plain) k_target_critic1<Rows32<1, true, 2, true>><<<grid, block, a > b ? a : b, s>>>(d, t, nt);
      else k_target_critic1<Rows32<1>><<<grid, block, a > b ? a : b, s>>>(d, t, nt);
    } else if (d.w2_plain) {
      k_target_critic1<Rows32<2, true, 2, true>><<<grid, block, a > b ? a : b, s>>>(d, t, nt);
    } else {
      k_target_critic1<Rows32<2>><<<grid, block, a > b ? a : b, s>>>(d, t, nt);
    }
    return hipGetLastError();
  }
  const dim3 grid(nt + nc), block(kThreads);
  if (!(d.rows_t == 16 && (d.rows_c == 64 || d.rows_c == 32)) && !(d.rows_t == d.rows_c && (d.rows_t == 32 || d.rows_t == 64)))
    return hipErrorInvalidValue;                     // the kernel exists for these row classes only
  if (d.actor_ahead && !(d.rows_t == 16 && d.rows_c == 32)) return hipErrorInvalidValue;
  if (d.rows_t == 16 && d.rows_c == 32) {
    const size_t a = chain_bytes<Rows16>(d.D, vec, Rows16::kStageForward), b = chain_bytes<Rows32<1>>(d.D, vec);
    if (d.actor_ahead) k_target_critic<Rows16, Rows32<1>, true><<<grid, block, Lds<1>(d.D).bytes(kAheadBase + ahead_floats<32>()), s>>>(d, t, nt);
    else k_target_critic<Rows16, Rows32<1>><<<grid, block, a > b ? a : b, s>>>(d, t, nt);
  } else if (d.rows_t == 16) {
    const size_t a = chain_bytes<Rows16>(d.D, vec, Rows16::kStageForward), b = chain_bytes<Rows32<2>>(d.D, vec);
    k_target_critic<Rows16, Rows32<2>><<<grid, block, a > b ? a : b, s>>>(d, t, nt);
  } else if (d.rows_t == 32) {
    k_target_critic<Rows32<1>, Rows32<1>><<<grid, block, chain_bytes<Rows32<1>>(d.D, vec), s>>>(d, t, nt);
  } else {
    k_target_critic<Rows64, Rows64><<<grid, dim3(Rows64::kThr), chain_bytes<Rows32<2>>(d.D, vec), s>>>(d, t, nt);
  }
  return hipGetLastError();
}
hipError_t launch_actor(const PopDev& d, uint32_t t, hipStream_t s) {
  const dim3 grid(xcd_grid(d.P, d.B / d.rows_a)), block(kThreads);
  const bool ahead = (d.spread & kSpreadActor) != 0;
  if ((d.actor_ahead || ahead) && d.rows_a != 16) return hipErrorInvalidValue;
  if (d.A > kMaxAct) {
    if (d.actor_ahead) return hipErrorInvalidValue;
    if (ahead) k_actor<Rows16Deep, 1, true, kSacMaxAct><<<grid, block, chain_bytes<Rows16>(d.D, vec_actor(d), Rows16::kStage, kWideScratch), s>>>(d, t);
    else if (d.rows_a == 16) k_actor<Rows16Deep, 1, false, kSacMaxAct><<<grid, block, chain_bytes<Rows16>(d.D, vec_actor(d), Rows16::kStage, kWideScratch), s>>>(d, t);
    else if (d.rows_a == 32) k_actor<Rows32Wide, 2, false, kSacMaxAct><<<grid, dim3(Rows32x8::kThr), chain_bytes<Rows32<1>>(d.D, vec_actor(d), Rows32<1>::kStage, kWideScratch), s>>>(d, t);
    else return hipErrorInvalidValue;
  } else if (d.D > kMaxIn) {
    if (d.actor_ahead) return hipErrorInvalidValue;
    if (ahead) k_actor<Rows16Deep, 1, true><<<grid, block, chain_bytes<Rows16>(d.D, vec_actor(d)), s>>>(d, t);
    else if (d.rows_a == 16) k_actor<Rows16Deep><<<grid, block, chain_bytes<Rows16>(d.D, vec_actor(d)), s>>>(d, t);
    else if (d.rows_a == 32) k_actor<Rows32Wide><<<grid, dim3(Rows32x8::kThr), chain_bytes<Rows32<1>>(d.D, vec_actor(d)), s>>>(d, t);
    else return hipErrorInvalidValue;
  } else if (d.actor_ahead || ahead) {
    if (d.w2_plain) k_actor<Rows16In<true>, 1, true><<<grid, block, chain_bytes<Rows16>(d.D, vec_actor(d)), s>>>(d, t);
    else k_actor<Rows16, 1, true><<<grid, block, chain_bytes<Rows16>(d.D, vec_actor(d)), s>>>(d, t);
  } else if (d.rows_a == 16 && d.w2_plain) k_actor<Rows16In<true>><<<grid, block, chain_bytes<Rows16>(d.D, vec_actor(d)), s>>>(d, t);
  else if (d.rows_a == 16) k_actor<Rows16><<<grid, block, chain_bytes<Rows16>(d.D, vec_actor(d)), s>>>(d, t);
  else if (d.rows_a == 32 && (int)grid.x > kCUs) k_actor<Rows32<1>, 2><<<grid, block, chain_bytes<Rows32<1>>(d.D, vec_actor(d)), s>>>(d, t);
  else if (d.rows_a == 32) k_actor<Rows32x8><<<grid, dim3(Rows32x8::kThr), chain_bytes<Rows32<1>>(d.D, vec_actor(d)), s>>>(d, t);
  else k_actor<Rows32<2>><<<grid, block, chain_bytes<Rows32<2>>(d.D, vec_actor(d)), s>>>(d, t);
  return hipGetLastError();
}
hipError_t launch_act_rows(const PopDev& d, const float* obs, int n, float* act, const float* sigma, const SigmaArgs* args, uint32_t step,
                           uint32_t row_base, int whole, hipStream_t s) {
  auto* kernel = sigma || args ? (d.w2_plain ? k_act<true, true> : k_act<false, true>) : (d.w2_plain ? k_act<true, false> : k_act<false, false>);
  const ActGrid g = act_grid(d.P, n);
  // Up to 16 outputs all four wavefronts share the head, unless rounds of workgroups each read another agent's weights, which then are on their way
  // from memory four times (us, shared / not: 512 agents 33 rows, 3 inputs, 37.0 / 38.2; 768 agents 5 rows 40.3 / 36.5, SAC of 6 actions 45.8 / 41.4; 512
  // agents 27.6 / 27.4).
  const int share_head = d.actor.out <= 16 && (whole > 32 || d.P <= kCUs);
  kernel<<<dim3(xcd_grid(d.P, g.chunks), g.pieces), dim3(kThreads), act_lds_bytes(d), s>>>(d, obs, n, act, sigma, step, row_base,
                                                                                                        g.chunks, share_head, args ? *args : kNoNoise);
  return hipGetLastError();
}

}  // namespace pop
