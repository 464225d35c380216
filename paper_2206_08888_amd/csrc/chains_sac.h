// Layer chains of the SAC update step (Sec. 4.1 of the paper names Soft Actor-Critic with the
// learned temperature, Haarnoja et al. 2018, next to TD3; same networks, same batch).
//
// The policy is a tanh-squashed diagonal Gaussian.  The actor MLP has 2A outputs,
//   (mu, ls) = actor(s), ls clamped to [-20, 2] (no gradient outside);
//   u = mu + exp(ls) eps, eps unit normal from the counter RNG;  a = tanh(u);
//   log pi(a|s) = sum_j [ -eps_j^2/2 - ls_j - ln(2 pi)/2 ] - sum_j 2 (ln 2 - u_j - softplus(-2 u_j)).
// One step, with alpha = exp(log_alpha) as it stands when the step starts:
//   sac_target_chain : a' ~ pi(.|s') from the ONLINE actor (stream 3), twin target critics,
//                      y = r + gamma (1 - d) (min_k Q'_k(s', a') - alpha log pi(a'|s'))
//   critic_chain     : the TD3 one, unchanged (chains.h)
//   sac_actor_chain  : a ~ pi(.|s) (stream 2), both updated critics on [s, a], per sample the
//                      gradient of -min_k Q_k flows through the smaller critic (the first on
//                      ties), plus alpha log pi; backward through the sampling into the actor
//   the temperature  : d/dlog_alpha of -alpha mean(log pi + target entropy), one Adam step on
//                      log_alpha in the actor's weight-gradient launch (wgrad.h)
// The critic targets move every step; there is no target actor and no delay.
#pragma once
#include "chains.h"

namespace pop {

namespace {

__device__ inline float softplusf(float x) { return fmaxf(x, 0.0f) + log1pf(expf(-fabsf(x))); }

constexpr float kLogStdMin = -20.0f, kLogStdMax = 2.0f;
constexpr float kHalfLog2Pi = 0.91893853320467274178f;
constexpr float kLn2 = 0.69314718055994530942f;

// Unit normal number `el` of stream `stream` at counter t (the update step's noise streams).
__device__ inline float normal_at(const HpDev& hp, uint32_t el, uint32_t t, uint32_t stream) {
  const U4 blk = philox4x32_10(hp.seed_lo, hp.seed_hi, el >> 2, t, stream, 0u);
  float n4[4];
  normals4(blk, n4);
  return (el & 2u) ? ((el & 1u) ? n4[3] : n4[2]) : ((el & 1u) ? n4[1] : n4[0]);
}

}  // namespace

// LDS scratch of the SAC chains: nine blocks of [R][kSs] floats (a block = kSacRegion of the
// map's [R][8] regions); the action dimension goes up to kSacMaxAct here.
constexpr int kSs = kSacMaxAct;
constexpr int kSacRegion = kSs / kMaxAct;
constexpr int kSacScratch = 9 * kSacRegion;
static_assert(kSs % kMaxAct == 0 && 2 * kSs >= kMaxHead, "dz3 rows of kMaxHead floats fit two scratch blocks");

// vectors the chains keep in LDS: the actor's head bias, the two critic heads and their biases (the wide
// operands -- the actor's head, the critics' first-layer rows of the action -- go through the matrix pipe
// straight from global memory)
constexpr int vec_sac_target_floats = kMaxHead + 2 * kH + 8;
inline int vec_sac_target(const PopDev&) { return vec_sac_target_floats; }
constexpr int vec_sac_actor_floats = kMaxHead + 2 * kH + 8;   // behind them: G::kStage floats for the products
inline int vec_sac_actor(const PopDev&) { return vec_sac_actor_floats; }

// ---------------------------------------------------------------------------------------------
// Target chain.  One workgroup per (agent, chunk).
// ONE: of the two target critics this workgroup runs number `one` only and publishes Q' - alpha log pi of each row (target_chain); the
// smaller of the two is that of the smaller Q', rounding included (and kInfMinusInf).
template <class G, bool ONE = false>
__device__ __forceinline__ void sac_target_chain(const PopDev& d, uint32_t t, int agent, int chunk, float* lds, int one = 0) {
  constexpr int R = G::R;
  const LdsMap<G::R, G::kPad> L(d.D, kSacScratch);
  const int A = d.A;
  float* Xs = lds;
  float* buf = lds + L.buf;
  float* hd = lds + L.s(0);                          // [R][kMaxHead]: means | log-stds (later the terms of log pi)
  float* qmin = lds + L.s(2 * kSacRegion);           // [R] min of the target critics, [R..2R) log pi
  float* v_ab3 = lds + L.vec;                        // [kMaxHead]
  float* v_cw3 = v_ab3 + kMaxHead;                   // [2][256]
  float* v_cb3 = v_cw3 + 2 * kH;                     // [2]
  float* stage = lds + L.vec + vec_sac_target_floats;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int r0 = chunk * R;
  const float* an = net_ptr(d, d.theta, agent, 0);   // the online actor: SAC has no target actor
  const float* tc0 = net_ptr(d, d.target, agent, 1 + (ONE ? one : 0));
  const float* tc1 = ONE ? tc0 : net_ptr(d, d.target, agent, 2);
  typename G::Pre pre;
  pre.load(an, d.actor, wave, lane);
  const HpDev hp = d.hp[agent];
  const float alpha = expf(d.log_alpha[agent]);
  const float* rows = batch_rows(d, t, agent) + (size_t)r0 * d.row;
  POP_MARK(0);
  if (d.D <= kMaxIn) {                               // one trip to memory for all of the prologue
    SmallVec ab3, cw3a, cw3b;
    InputTile<R, G::kThr> xin;
    ab3.fetch(an + d.actor.b3, 2 * A, tid);
    cw3a.fetch(tc0 + d.critic.w3, kH, tid);
    cw3b.fetch(tc1 + d.critic.w3, kH, tid);
    const float cb3 = (tid == 0 ? tc0 : tc1)[d.critic.b3];
    xin.fetch(L.xld, rows, d.row, d.D + 2, d.O, R, tid);
    ab3.put(v_ab3, 2 * A, tid);
    cw3a.put(v_cw3, kH, tid);
    cw3b.put(v_cw3 + kH, kH, tid);
    if (tid < 2) v_cb3[tid] = cb3;
    xin.put(Xs, L.xld, tid);
  } else {
    stage_vector<G::kThr>(v_ab3, an + d.actor.b3, 2 * A, tid);
    stage_vector<G::kThr>(v_cw3, tc0 + d.critic.w3, kH, tid);
    stage_vector<G::kThr>(v_cw3 + kH, tc1 + d.critic.w3, kH, tid);
    if (tid < 2) v_cb3[tid] = (tid == 0 ? tc0 : tc1)[d.critic.b3];
    G::load_input(Xs, L.xld, rows, d.row, d.D + 2, d.O, R, tid);
  }
  __syncthreads();
  POP_MARK(1);

  G::template first_layer<false>(Xs, L.xld, an, d.actor, pre, buf, nullptr, wave, lane, stage);
  __syncthreads();
  POP_MARK(2);
  G::template hidden_layer<false>(buf, an, d.actor, pre, nullptr, wave, lane, [&]() { pre.load(tc0, d.critic, wave, lane); }, stage);
  __syncthreads();
  POP_MARK(3);
  if (G::kStage > 0 && 2 * A <= 16) head_split<G, false>(buf, an + d.actor.w3, 2 * A, hd, kMaxHead, wave, lane, stage);
  else head_mfma<R, G::kThr>(buf, an + d.actor.w3, 2 * A, hd, kMaxHead, wave, lane);
  __syncthreads();
  POP_MARK(4);
  for (int e = tid; e < R * A; e += G::kThr) {
    const int r = e / A, j = e - r * A;
    const float mu = hd[r * kMaxHead + j] + v_ab3[j];
    const float ls = fminf(fmaxf(hd[r * kMaxHead + A + j] + v_ab3[A + j], kLogStdMin), kLogStdMax);
    const float eps = normal_at(hp, (uint32_t)((r0 + r) * A + j), t, kStreamSacS2);
    const float u = mu + expf(ls) * eps;
    Xs[r * L.xld + d.O + j] = tanhf(u);
    hd[r * kMaxHead + A + j] = -0.5f * eps * eps - ls - kHalfLog2Pi - 2.0f * (kLn2 - u - softplusf(-2.0f * u));
  }
  __syncthreads();
  if (tid < R) {
    float lp = 0.0f;
    for (int j = 0; j < A; ++j) lp += hd[tid * kMaxHead + A + j];
    qmin[R + tid] = lp;
  }
  POP_MARK(5);

#pragma unroll
  for (int k = 0; k < (ONE ? 1 : 2); ++k) {
    const float* tc = k == 0 ? tc0 : tc1;
    G::template first_layer<false>(Xs, L.xld, tc, d.critic, pre, buf, nullptr, wave, lane, stage);
    __syncthreads();
    POP_MARK(6 + 3 * k);
    G::template hidden_layer<false>(buf, tc, d.critic, pre, nullptr, wave, lane,
                                    [&]() { if (!ONE && k == 0) pre.load(tc1, d.critic, wave, lane); }, stage);
    __syncthreads();
    POP_MARK(7 + 3 * k);
    G::thin(buf, v_cw3 + k * kH, 1, hd, tid, kMaxHead);
    __syncthreads();
    if (tid < R) {
      const float q = hd[tid * kMaxHead] + v_cb3[k];
      qmin[tid] = k == 0 ? q : fminf(qmin[tid], q);
    }
    __syncthreads();
    POP_MARK(8 + 3 * k);
  }
  if (ONE) {
    if (tid < R) {
      const float q = qmin[tid], v = q - alpha * qmin[R + tid];
      publish_y(d, ((size_t)one * d.P + agent) * d.B + r0 + tid, t, q == -INFINITY && v != v ? __uint_as_float(kInfMinusInf) : v);
    }
  } else if (tid < R) {
    const float rew = rows[(size_t)tid * d.row + d.D];
    const float done = rows[(size_t)tid * d.row + d.D + 1];
    const float yv = rew + hp.gamma * (1.0f - done) * (qmin[tid] - alpha * qmin[R + tid]);
    d.y[(size_t)agent * d.B + r0 + tid] = yv;
    publish_y(d, (size_t)agent * d.B + r0 + tid, t, yv);
  }
  POP_MARK(12);
}

// Backward through the actor's head for one chunk, thread c = hidden unit c:
//   gW3[c][j] = sum_r h2[r][c] dz3[r][j];  dz2[r][c] = [h2[r][c] > 0] sum_j dz3[r][j] W3[c][j]
// buf: h2 in, dz2 out (LDS tile, row stride kLda); dz3: [R][kMaxHead], columns >= H2 hold zeros; W3: the
// head's weights [256][H2];
// NC: head columns handled (a multiple of 4, >= H2).
// w3: the unit's row of the head's weights, requested ahead by sac_head_row in pairs (H2 is even, a row 8-byte aligned): a lane's
// row lies H2 floats from its neighbour's, so that a load touches up to 64 cache lines whatever its width.
template <int NC>
__device__ __forceinline__ void sac_head_row(f32x2 (&w3)[NC / 2], const float* __restrict__ W3, int H2, int c) {
#pragma unroll
  for (int j = 0; j < NC / 2; ++j) {
    w3[j] = f32x2{0.0f, 0.0f};
    if (2 * j < H2) w3[j] = *reinterpret_cast<const f32x2*>(W3 + c * H2 + 2 * j);
  }
}
template <class G, int NC>
__device__ __forceinline__ void sac_head_backward(float* buf, const float* dz3, const f32x2 (&w3)[NC / 2], int H2,
                                                  float* zg, float* part, float* cross, int tid) {
  using UR = UnitRows<G>;
  const int c = tid & (kH - 1);
  float sums[UR::kOwn][NC + 1];                      // dW3 by column, db2
#pragma unroll
  for (int o = 0; o < UR::kOwn; ++o)
#pragma unroll
    for (int j = 0; j <= NC; ++j) sums[o][j] = 0.0f;
  zg += c;
  constexpr int RB = NC <= 16 ? 4 / UR::kOwn : 1;    // rows of a half in flight
#pragma unroll 1
  for (int rb = 0; rb < UR::kRows; rb += RB) {
#pragma unroll
    for (int o = 0; o < UR::kOwn; ++o)
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        const int r = UR::row0(o, tid) + rb + i;
        const float h = buf[r * kLda + c];
        float dh = 0.0f;
#pragma unroll
        for (int q = 0; q < NC / 4; ++q) {
          const f32x4 g = *reinterpret_cast<const f32x4*>(&dz3[r * kMaxHead + 4 * q]);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            sums[o][4 * q + k] += h * g[k];
            dh += g[k] * w3[2 * q + (k >> 1)][k & 1];
          }
        }
        const float z = h > 0.0f ? dh : 0.0f;
        buf[r * kLda + c] = z;
        zg[r * kH] = z;
        sums[o][NC] += z;
      }
  }
  // the halves' sums meet, as many columns at a time as the slabs hold
  constexpr int CH = UR::kCross ? (G::kStage / kH < NC + 1 ? G::kStage / kH : NC + 1) : NC + 1;
#pragma unroll
  for (int j0 = 0; j0 <= NC; j0 += CH) {
    if (UR::kCross) {
      if (j0) __syncthreads();
      if (tid >= kH) {
#pragma unroll
        for (int j = j0; j <= NC && j < j0 + CH; ++j) cross[(j - j0) * kH + c] = sums[0][j];
      }
      __syncthreads();
    }
    if (tid < kH) {
#pragma unroll
      for (int j = j0; j <= NC && j < j0 + CH; ++j) {
        const float v = UR::kCross ? sums[0][j] + cross[(j - j0) * kH + c] : UR::kHalves == 1 ? sums[0][j] : sums[0][j] + sums[UR::kOwn - 1][j];
        if (j == NC) part[kAP_db2 + c] = v;
        else if (j < H2) part[kAP_dW3 + j * kH + c] = v;
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Actor chain.  One workgroup per (agent, chunk).
//   L = (1/B) sum_b [ alpha log pi(a_b|s_b) - min_k Q_k(s_b, a_b) ]
//   critic k (k = the smaller one for that sample): dz2 = -(1/B) W3^T * [h2 > 0]; dz1 = (dz2 W2^T) * [h1 > 0];
//             da += dz1 W1[O:O+A, :]^T
//   sampling:  du = da (1 - a^2) + (alpha/B) 2a;  dmu = du;  dls = (du std eps - alpha/B) * [ls inside its range]
//   actor:     dz3 = [dmu, dls]; dz2 = (dz3 W3^T) * [h2 > 0]; dz1 = (dz2 W2^T) * [h1 > 0]
template <class G>
__device__ __forceinline__ void sac_actor_chain(const PopDev& d, uint32_t t, int agent, int chunk, float* lds) {
  constexpr int R = G::R;
  const LdsMap<G::R, G::kPad> L(d.D, kSacScratch);
  const int A = d.A, H2 = 2 * d.A;
  float* Xs = lds;
  float* buf = lds + L.buf;
  float* hd = lds + L.s(0);                          // [R][kMaxHead]: means -> terms of log pi -> thin-product scratch
                                                     //                | log-stds -> std * eps
  float* ap = lds + L.s(2 * kSacRegion);             // a = tanh(u)
  float* ins = lds + L.s(3 * kSacRegion);            // 1 where the log-std was inside its range
  float* qv = lds + L.s(4 * kSacRegion);             // [R] q1 | q2 | seed1 | seed2 | log pi
  float* da1 = lds + L.s(5 * kSacRegion);
  float* da2 = lds + L.s(6 * kSacRegion);
  float* dz3 = lds + L.s(7 * kSacRegion);            // [R][kMaxHead] (two blocks)
  float* v_ab3 = lds + L.vec;                        // [kMaxHead]
  float* v_cw3 = v_ab3 + kMaxHead;                   // [2][256] critic heads
  float* v_cb3 = v_cw3 + 2 * kH;                     // [2]
  float* stage = lds + L.vec + vec_sac_actor_floats;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int r0 = chunk * R;
  const HpDev hp = d.hp[agent];
  const float alpha = expf(d.log_alpha[agent]);
  const float invB = 1.0f / (float)d.B;
  const float* an = net_ptr(d, d.theta, agent, 0);
  const float* cn[2] = {net_ptr(d, d.theta, agent, 1), net_ptr(d, d.theta, agent, 2)};
  typename G::Pre pre;
  pre.load(an, d.actor, wave, lane);
  const float* rows = batch_rows(d, t, agent) + (size_t)r0 * d.row;
  const size_t act_off = ((size_t)agent * d.B + r0) * kH;
  float* part = d.apart + ((size_t)agent * (d.B / R) + chunk) * kAPart;
  POP_MARK(20);
  if (d.D <= kMaxIn) {                               // one trip to memory for all of the prologue
    SmallVec ab3, cw3a, cw3b;
    InputTile<R, G::kThr> xin;
    ab3.fetch(an + d.actor.b3, H2, tid);
    cw3a.fetch(cn[0] + d.critic.w3, kH, tid);
    cw3b.fetch(cn[1] + d.critic.w3, kH, tid);
    const float cb3 = (tid == 0 ? cn[0] : cn[1])[d.critic.b3];
    xin.fetch(L.xld, rows, d.row, 0, d.O, R, tid);
    ab3.put(v_ab3, H2, tid);
    cw3a.put(v_cw3, kH, tid);
    cw3b.put(v_cw3 + kH, kH, tid);
    if (tid < 2) v_cb3[tid] = cb3;
    xin.put(Xs, L.xld, tid);
  } else {
    stage_vector<G::kThr>(v_ab3, an + d.actor.b3, H2, tid);
    for (int k = 0; k < 2; ++k) stage_vector<G::kThr>(v_cw3 + k * kH, cn[k] + d.critic.w3, kH, tid);
    if (tid < 2) v_cb3[tid] = cn[tid][d.critic.b3];
    G::load_input(Xs, L.xld, rows, d.row, 0, d.O, R, tid);
  }
  __syncthreads();
  POP_MARK(21);

  const uint64_t mask_a1 = G::template first_layer<false>(Xs, L.xld, an, d.actor, pre, buf, d.aH1 + act_off, wave, lane, stage);
  __syncthreads();
  G::template hidden_layer<false>(buf, an, d.actor, pre, d.aH2 + act_off, wave, lane,
                                  [&]() { pre.load(cn[0], d.critic, wave, lane); }, stage);
  __syncthreads();
  POP_MARK(22);
  if (G::kStage > 0 && H2 <= 16) head_split<G, false>(buf, an + d.actor.w3, H2, hd, kMaxHead, wave, lane, stage);
  else head_mfma<R, G::kThr>(buf, an + d.actor.w3, H2, hd, kMaxHead, wave, lane);
  __syncthreads();
  for (int e = tid; e < R * A; e += G::kThr) {
    const int r = e / A, j = e - r * A, o = r * kSs + j, om = r * kMaxHead + j, ol = om + A;
    const float mu = hd[om] + v_ab3[j];
    const float ls_raw = hd[ol] + v_ab3[A + j];
    const float ls = fminf(fmaxf(ls_raw, kLogStdMin), kLogStdMax);
    const float eps = normal_at(hp, (uint32_t)((r0 + r) * A + j), t, kStreamSacS);
    const float se = expf(ls) * eps;
    const float u = mu + se;
    const float a = tanhf(u);
    ap[o] = a;
    Xs[r * L.xld + d.O + j] = a;
    hd[ol] = se;
    ins[o] = (ls_raw >= kLogStdMin && ls_raw <= kLogStdMax) ? 1.0f : 0.0f;
    hd[om] = -0.5f * eps * eps - ls - kHalfLog2Pi - 2.0f * (kLn2 - u - softplusf(-2.0f * u));
  }
  __syncthreads();
  if (tid < R) {
    float lp = 0.0f;
    for (int j = 0; j < A; ++j) lp += hd[tid * kMaxHead + j];
    qv[4 * R + tid] = lp;
  }
  POP_MARK(23);

  // both critics forward on [s, a]; the ReLU patterns of both layers stay in registers
  uint64_t mask1[2], mask2[2];
  typename G::WtBlock wt;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    mask1[k] = G::template first_layer<false>(Xs, L.xld, cn[k], d.critic, pre, buf, nullptr, wave, lane, stage);
    __syncthreads();
    mask2[k] = G::template hidden_layer<false>(buf, cn[k], d.critic, pre, nullptr, wave, lane, [&]() {
      if (k == 0) pre.load(cn[1], d.critic, wave, lane);
      else G::load_wt(wt, cn[0] + d.critic.w2, wave, lane);
    }, stage);
    __syncthreads();
    G::thin(buf, v_cw3 + k * kH, 1, hd, tid, kMaxHead);
    __syncthreads();
    if (tid < R) qv[k * R + tid] = hd[tid * kMaxHead] + v_cb3[k];
    __syncthreads();
    POP_MARK(24 + k);
  }
  if (tid < 64) {                                    // R <= 64: one wavefront covers the chunk
    float term = 0.0f, lp = 0.0f;
    if (tid < R) {
      const float q1 = qv[tid], q2 = qv[R + tid];
      const bool first = q1 <= q2;                   // ties go to the first critic
      qv[2 * R + tid] = first ? -invB : 0.0f;
      qv[3 * R + tid] = first ? 0.0f : -invB;
      lp = qv[4 * R + tid];
      term = alpha * lp - (first ? q1 : q2);
    }
    const float s_loss = wave_sum(term), s_lp = wave_sum(lp);
    if (tid == 0) { part[kAP_loss] = s_loss * invB; part[kAP_logp] = s_lp; }
  }
  __syncthreads();

  // both critics backward to the action
  constexpr int W = G::kThr / 64;                    // wavefronts
  f32x4 h2r[R / W];                                  // this thread's share of the actor's parked h2 tile
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    G::store_outer_masked(buf, mask2[k], qv + (2 + k) * R, v_cw3 + k * kH, wave, lane);     // dz2 of critic k
    __syncthreads();
    const float* h2g = d.aH2 + act_off;
    G::input_grad_to_lds(buf, cn[k] + d.critic.w2, wt, mask1[k], wave, lane, [&]() {
      if (k == 0) return;
#pragma unroll
      for (int i = 0; i < R / W; ++i)
        h2r[i] = *reinterpret_cast<const f32x4*>(h2g + (W * i + (tid >> 6)) * kH + 4 * (tid & 63));
    }, stage);                                       // buf = dz1 of critic k
    __syncthreads();
    if (G::kStage > 0 && A <= 16) head_split<G, true>(buf, cn[k] + d.critic.w1 + d.O * kH, A, k == 0 ? da1 : da2, kSs, wave, lane, stage);
    else head_mfma_t<R, G::kThr>(buf, cn[k] + d.critic.w1 + d.O * kH, A, k == 0 ? da1 : da2, kSs, wave, lane);
    if (k == 0) G::load_wt(wt, cn[1] + d.critic.w2, wave, lane);
    else G::load_wt(wt, an + d.actor.w2, wave, lane);
    __syncthreads();
    POP_MARK(26 + k);
  }

  // through the sampling into the actor's head and back through it, a thread per hidden unit; NC columns in registers
  const float ab = alpha * invB;
  float* cross = stage;                              // the slabs are idle here
  auto head_back = [&](auto NC_) {
    constexpr int NC = decltype(NC_)::value;
    f32x2 w3[NC / 2];
    sac_head_row<NC>(w3, an + d.actor.w3, H2, tid & (kH - 1));
    for (int e = tid; e < R * kMaxHead; e += G::kThr) {
      const int r = e / kMaxHead, c = e - r * kMaxHead;
      float g = 0.0f;
      if (c < H2) {
        const int j = c < A ? c : c - A, o = r * kSs + j;
        const float a = ap[o];
        const float du = (da1[o] + da2[o]) * (1.0f - a * a) + ab * 2.0f * a;
        g = c < A ? du : (du * hd[r * kMaxHead + A + j] - ab) * ins[o];
      }
      dz3[e] = g;                                      // unused columns are kept at zero
    }
#pragma unroll
    for (int i = 0; i < R / W; ++i)                    // h2 of the actor back into the tile
      *reinterpret_cast<f32x4*>(&buf[(W * i + (tid >> 6)) * kLda + 4 * (tid & 63)]) = h2r[i];
    __syncthreads();
    if (tid < H2) {
      float s = 0.0f;
#pragma unroll 16
      for (int r = 0; r < R; ++r) s += dz3[r * kMaxHead + tid];
      part[kAP_db3 + tid] = s;
    }
    POP_MARK(28);
    sac_head_backward<G, NC>(buf, dz3, w3, H2, d.adZ2 + act_off, part, cross, tid);
  };
  if (H2 <= 16) head_back(IntC<16>());
  else if (H2 <= 36) head_back(IntC<36>());
  else head_back(IntC<kMaxHead>());
  __syncthreads();
  POP_MARK(29);
  G::template input_grad_to_global<false>(buf, an + d.actor.w2, wt, mask_a1, d.adZ1 + act_off, part + kAP_db1, wave, lane, stage);
  POP_MARK(30);
}

}  // namespace pop
