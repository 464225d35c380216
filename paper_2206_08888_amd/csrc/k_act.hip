// Acting on a few observations per agent (one environment step, evaluation with a handful of environments):
// obs -> actor, one workgroup of sixteen wavefronts per agent and RR observations.
//
// One row is 66,000 multiply-adds per agent against 256 KB of W2, so the kernel is the trip of those weights to the CU and what
// stands before and behind it.  The whole of W2 is requested at the start into registers (64 per lane: wavefront w has the rows
// 16 w .. 16 w + 15, lane l the columns 4 l ..), and the first layer runs under that trip.  Each wavefront contracts over its
// own 16 rows on the vector ALU (256 instructions per lane and observation row; 4x4x1 matrix instructions would take the time of four rows for one),
// and the sixteen partial sums meet in LDS: rounding steps per sum 16 + 16 where a 256-deep chain has 256.
// The 32-row workgroups of k_act spend 8 us on the same, most of it on rows that are not there; with many agents, rows or outputs they are ahead
// all the same (most_agents).
#include "chains.h"

namespace pop {

constexpr int kFewWaves = 16, kFewThr = 64 * kFewWaves;

template <int RR>
struct FewMap {                            // LDS (floats): observations | partial sums | hidden layer | head sums | head weights
  static constexpr int kObsLd = kSacMaxIn;
  static constexpr int obs = 0, part = RR * kObsLd, hidden = part + kFewWaves * RR * kH, head = hidden + RR * kH,
                       w3 = head + RR * kMaxHead;
  __host__ __device__ static constexpr int w3_ld(int J) { return J | 1; }   // a hidden unit's weights: odd, four lanes to a bank at most
  static constexpr size_t bytes(int J) { return sizeof(float) * (w3 + (J ? kH * w3_ld(J) : 0)); }   // J = 0: no head weights
};

// WIDE: more than 64 inputs.  Below that the first-layer weights are one batch of loads per lane.
// LINES: a head of many columns.  A column requested by its wavefront is a line per lane, and more than one or two of those keep the load path busy longer
// than k_act takes for all of it; whole lines take a detour through LDS.  us per call, 17 inputs 1 row, columns / lines: 48 outputs 11.1 / 7.9 with 80 agents,
// 16.6 / 13.8 with 200; 24 outputs 8.3 / 7.0 and 13.1 / 12.2; 6 outputs 6.6 / 6.6 with 64, 11.4 / 11.6 with 200; 376 inputs, 17 outputs: 17.1 / 15.9 with 128, 27.5 /
// 27.8 with 256.
template <int RR, bool PLAIN, bool WIDE, bool LINES>
__global__ __launch_bounds__(kFewThr) void k_act_few(PopDev d, const float* __restrict__ obs, int n, float* __restrict__ act,
                                                     const float* __restrict__ sigma, SigmaArgs sigma_args, uint32_t step, uint32_t row_base) {
  warm_args<sizeof(PopDev) + 32>();
  asm volatile("" ::"s"(step), "s"(row_base));
  extern __shared__ __attribute__((aligned(16))) float lds[];
  using L = FewMap<RR>;
  float* xs = lds + L::obs;
  float* part = lds + L::part;
  float* hid = lds + L::hidden;
  float* head = lds + L::head;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int agent, chunk;
  if (!decode_block(blockIdx.x, d.P, (n + RR - 1) / RR, agent, chunk)) return;
  const int r0 = chunk * RR, valid = n - r0 < RR ? n - r0 : RR;
  const int K = d.O, A = d.A, J = d.actor.out;       // SAC: 2 A outputs, the means come first
  const float* an = net_ptr(d, d.theta, agent, 0);
  // observations first, then the first layer's weights, then W2: a wavefront's loads come back in the order they went out
  const float* rows = obs + ((size_t)agent * n + r0) * K;
  constexpr int XI = (RR * L::kObsLd + kFewThr - 1) / kFewThr;
  float xv[XI];
#pragma unroll
  for (int i = 0; i < XI; ++i) {
    const int e = tid + i * kFewThr;
    xv[i] = 0.0f;
    if (e < valid * K) xv[i] = rows[e];
  }
  constexpr int U = 4;                               // rows of W1 per wavefront and batch: k = 64 b + 16 u + wave
  auto load_w1 = [&](f32x4 (&w)[U], int b) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = 64 * b + 16 * u + wave;
      w[u] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      if (k < K) w[u] = *reinterpret_cast<const f32x4*>(an + d.actor.w1 + (size_t)k * kH + 4 * lane);
    }
  };
  f32x4 w1[U];
  load_w1(w1, 0);
  f32x4 w2[16];
  auto load_w2 = [&]() {
    const float* p = an + d.actor.w2 + w2_index<PLAIN>(16 * wave, 0) + w2_index<PLAIN>(0, 4 * lane);
#pragma unroll
    for (int i = 0; i < 16; ++i) w2[i] = *reinterpret_cast<const f32x4*>(p + w2_index<PLAIN>(i, 0));
  };
  const int nb = (K + 63) / 64;
  // The head's weights: the wavefront's columns wave, wave + 16, wave + 32 of the hidden units 4 lane .., or (LINES) whole lines on their way to LDS
  constexpr int JQ = kMaxHead / kFewWaves, W3I = kMaxHead * kH / 4 / kFewThr;
  float w3[LINES ? 1 : JQ][4];
  f32x4 w3_lines[LINES ? W3I : 1];
  if constexpr (LINES) {
#pragma unroll
    for (int i = 0; i < W3I; ++i) {
      const int e = tid + i * kFewThr;
      w3_lines[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      if (e < J * (kH / 4)) w3_lines[i] = *reinterpret_cast<const f32x4*>(an + d.actor.w3 + 4 * e);
    }
  } else {
#pragma unroll
    for (int q = 0; q < JQ; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        w3[q][e] = 0.0f;
        if (wave + kFewWaves * q < J) w3[q][e] = an[d.actor.w3 + (4 * lane + e) * J + wave + kFewWaves * q];
      }
  }
  // biases of the sums this thread adds up
  const float b1 = an[d.actor.b1 + (tid & (kH - 1))], b2 = an[d.actor.b2 + (tid & (kH - 1))];
  // what the last step needs: thread e has action j of row r, its head biases and its noise
  const int r_out = tid / A, j_out = tid - r_out * A;
  const bool last = tid < valid * A;
  const float ab3 = last ? an[d.actor.b3 + j_out] : 0.0f;
  const bool sac = d.algo == 1;
  const float lb3 = last && sac ? an[d.actor.b3 + A + j_out] : 0.0f;
  const float sg = sigma ? sigma[agent] : sigma_args.s[agent < kStaticMaxP ? agent : 0];
  if (!WIDE) load_w2();
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < XI; ++i) {                     // rows of K floats lie one behind the other here as well; rows past the last hold zeros
    const int e = tid + i * kFewThr;
    if (e < RR * L::kObsLd) xs[e] = xv[i];
  }
  __syncthreads();

  f32x4 acc[RR];
  auto sum_w1 = [&](const f32x4 (&w)[U], int b) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = 64 * b + 16 * u + wave;
      if (k < K) {
#pragma unroll
        for (int r = 0; r < RR; ++r) acc[r] += xs[r * K + k] * w[u];
      }
    }
  };
  // the partial sums of the wavefronts, in their order, and the layer's bias and ReLU
  auto meet = [&](float bias) {
#pragma unroll
    for (int r = 0; r < RR; ++r) *reinterpret_cast<f32x4*>(part + (wave * RR + r) * kH + 4 * lane) = acc[r];
    __syncthreads();
    if (tid < RR * kH) {
      float s[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        s[q] = part[4 * q * RR * kH + tid];
#pragma unroll
        for (int i = 1; i < 4; ++i) s[q] += part[(4 * q + i) * RR * kH + tid];
      }
      hid[tid] = fmaxf(((s[0] + s[1]) + (s[2] + s[3])) + bias, 0.0f);
    }
    __syncthreads();
  };
#pragma unroll
  for (int r = 0; r < RR; ++r) acc[r] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  if (WIDE) {
#pragma unroll 1
    for (int b = 0; b + 1 < nb; ++b) {
      f32x4 next[U];
      load_w1(next, b + 1);
      __builtin_amdgcn_sched_barrier(0);
      sum_w1(w1, b);
#pragma unroll
      for (int u = 0; u < U; ++u) w1[u] = next[u];
    }
    load_w2();
    __builtin_amdgcn_sched_barrier(0);
  }
  sum_w1(w1, nb - 1);
  meet(b1);

  float* w3l = lds + L::w3;
  const int ld3 = L::w3_ld(J);
  if constexpr (LINES) {                             // to LDS while W2 arrives, read behind the next barriers
    const float inv = 1.0f / (float)J;
#pragma unroll
    for (int i = 0; i < W3I; ++i) {
      const int e = 4 * (tid + i * kFewThr);
      if (e < J * kH) {
#pragma unroll
        for (int k = 0; k < 4; ++k) w3l[e + k + (ld3 - J) * (int)(((float)(e + k) + 0.5f) * inv)] = w3_lines[i][k];   // unit (e + k) / J, as in gather_run
      }
    }
  }
  float nz = 0.0f;                                   // drawn while W2 arrives
  if (sg > 0.0f && last) {
    const HpDev hp = d.hp[agent];
    const uint32_t el = (row_base + (uint32_t)(r0 + r_out)) * (uint32_t)A + (uint32_t)j_out;
    const U4 blk = philox4x32_10(hp.seed_lo, hp.seed_hi, el >> 2, step, kStreamExplore, 0u);
    float n4[4];
    normals4(blk, n4);
    nz = (el & 2u) ? ((el & 1u) ? n4[3] : n4[2]) : ((el & 1u) ? n4[1] : n4[0]);
  }
#pragma unroll
  for (int r = 0; r < RR; ++r) {
    acc[r] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 h = *reinterpret_cast<const f32x4*>(hid + r * kH + 16 * wave + 4 * q);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[r] += h[e] * w2[4 * q + e];
    }
  }
  meet(b2);
#pragma unroll
  for (int q = 0; q < JQ; ++q) {
    if (wave + kFewWaves * q < J) {
      float w[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if constexpr (LINES) w[e] = w3l[(4 * lane + e) * ld3 + wave + kFewWaves * q];
        else w[e] = w3[q][e];
      }
#pragma unroll
      for (int r = 0; r < RR; ++r) {
        const f32x4 h = *reinterpret_cast<const f32x4*>(hid + r * kH + 4 * lane);
        const float s = wave_sum((h[0] * w[0] + h[1] * w[1]) + (h[2] * w[2] + h[3] * w[3]));
        if (lane == 0) head[r * kMaxHead + wave + kFewWaves * q] = s;
      }
    }
  }
  __syncthreads();
  if (last) {
    const float pre_act = head[r_out * kMaxHead + j_out] + ab3;
    float a = tanhf(pre_act);
    if (sg > 0.0f) {
      if (sac) {                                     // a sample of the policy itself, its std scaled by sigma
        const float ls = fminf(fmaxf(head[r_out * kMaxHead + A + j_out] + lb3, -20.0f), 2.0f);
        a = tanhf(pre_act + sg * expf(ls) * nz);
      } else {
        a = fminf(fmaxf(a + sg * nz, -1.0f), 1.0f);
      }
    }
    act[((size_t)agent * n + r0 + r_out) * A + j_out] = a;
  }
}

namespace {
template <int RR, bool PLAIN, bool WIDE>
const void* few_kernel(bool lines) { return lines ? (const void*)k_act_few<RR, PLAIN, WIDE, true> : (const void*)k_act_few<RR, PLAIN, WIDE, false>; }
template <int RR>
const void* few_kernel(bool plain, bool wide, bool lines) {
  return plain ? (wide ? few_kernel<RR, true, true>(lines) : few_kernel<RR, true, false>(lines))
               : (wide ? few_kernel<RR, false, true>(lines) : few_kernel<RR, false, false>(lines));
}
template <int RR>
hipError_t setup_few() {
  for (int form = 0; form < 8; ++form) {
    const hipError_t e = hipFuncSetAttribute(few_kernel<RR>(form & 1, form & 2, form & 4), hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)FewMap<RR>::bytes(form & 4 ? kMaxHead : 0));
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}
template <int RR>
hipError_t launch_few(const PopDev& d, const float* obs, int n, float* act, const float* sigma, const SigmaArgs* args, uint32_t step,
                      uint32_t row_base, hipStream_t s) {
  const int J = d.actor.out;
  const bool lines = J >= kFewWaves + 4 || (J > kFewWaves && d.P <= kCUs / 2);
  using Kernel = void (*)(PopDev, const float*, int, float*, const float*, SigmaArgs, uint32_t, uint32_t);
  auto kernel = (Kernel)few_kernel<RR>(d.w2_plain != 0, d.O > 64, lines);
  kernel<<<dim3(xcd_grid(d.P, (n + RR - 1) / RR)), dim3(kFewThr), FewMap<RR>::bytes(lines ? J : 0), s>>>(d, obs, n, act, sigma, args ? *args : kNoNoise, step,
                                                                                                         row_base);
  return hipGetLastError();
}
}  // namespace

hipError_t setup_act_kernels() {
  hipError_t e;
  if ((e = setup_few<1>()) != hipSuccess || (e = setup_few<2>()) != hipSuccess) return e;
  return setup_few<4>();
}

// One workgroup of sixteen wavefronts fills a CU's registers.  As long as every RR rows get a CU to themselves the fewest rows per
// workgroup end soonest; up to four rows per agent they are ahead of k_act's 32-row workgroups with more agents too (most_agents).
// us per call with exploration noise, k_act behind a launch for the noise scales / here: 10 agents 1 row 14.6 / 8.0 (the host's share: 8), 50 rows 14.7 / 8.1,
// 256 agents 1 row 18.5 / 13.5, 4 rows 18.6 / 15.5, 80 agents 8 rows 15.2 / 10.6; 376 inputs: 10 agents 1 row 33.2 / 10.9, 40 rows 37.3 / 12.4, 80
// agents 1 row 42.0 / 15.1.
namespace {
// The most agents with which workgroups of RR rows are ahead of k_act, which reads an agent's weights once for all of its rows and has a head of
// matrix instructions, but spends a row block's time on one row and reads the first layer's weights block after block: the fewer rows here, the fewer
// outputs and the more inputs, the longer this kernel stays ahead.  us, k_act / here, without noise:
//   17 inputs, 6 outputs: 1 row 52.0 / 48.6 with 1024 agents, 110.5 / 107.8 with 2048; 2 rows 26.5 / 25.9 with 512, 52.5 / 52.7 with 1024; 3 rows 23.3 / 23.0 with
//   304, 23.5 / 24.0 with 384
//   12 and 16 outputs: 17 inputs 12 outputs, 3 rows, 22.7 / 23.4 with 257; 3 inputs 16 outputs, 1 row the same with 768, 4 % longer with 1024, 2 rows 1 % longer with 384
//   17 inputs, 48 outputs: 1 row 18.4 / 16.2 with 256, 30.8 / 31.0 with 512; 2 rows 18.4 / 17.8 with 256, 27.5 / 28.6 with 384; 4 rows 15.0 / 12.4 with 128, 15.3 /
//   15.6 with 136; 8 rows 15.0 / 14.7 with 120, 15.2 / 15.5 with 128
//   65 inputs, 3 rows: 8 outputs 27.4 / 24.7 with 257, 137.5 / 136.4 with 2048; 12 outputs 28.2 / 28.0 with 384, 32.4 / 32.5 with 512; 16 outputs 27.1 / 27.2
//   with 257; 48 outputs, 2 rows, 5 % shorter with 768, 1 % longer with 1024
int64_t most_agents(int RR, int rows, int inputs, int outputs) {
  constexpr int64_t any = 1 << 24;
  if (inputs > 64) {
    if (RR == 1 || inputs >= 256) return any;
    if (RR == 2) return outputs <= 32 || inputs >= 128 ? any : 768;
    if (outputs <= 8 || (outputs <= 16 && inputs >= 96)) return any;
    return outputs <= 12 ? 384 : 256;
  }
  if (outputs <= 8) return RR == 1 ? 2048 : RR == 2 ? 512 : 304;
  if (outputs <= 16) return RR == 1 ? 768 : RR == 2 ? 384 : 256;
  return RR == 1 ? 448 : RR == 2 ? 256 : rows <= 4 ? 128 : 120;
}
}  // namespace
hipError_t launch_act(const PopDev& d, const float* obs, int n, float* act, const float* sigma, const SigmaArgs* args, uint32_t step,
                      uint32_t row_base, int whole, hipStream_t s) {
  const auto ahead = [&](int RR) {
    return (whole <= RR || (int64_t)d.P * (((int64_t)whole + RR - 1) / RR) <= kCUs) && d.P <= most_agents(RR, whole, d.O, d.actor.out);
  };
  if (ahead(1)) return launch_few<1>(d, obs, n, act, sigma, args, step, row_base, s);
  if (ahead(2)) return launch_few<2>(d, obs, n, act, sigma, args, step, row_base, s);
  if (ahead(4)) return launch_few<4>(d, obs, n, act, sigma, args, step, row_base, s);
  return launch_act_rows(d, obs, n, act, sigma, args, step, row_base, whole, s);
}

}  // namespace pop
