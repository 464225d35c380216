// Replay sample + gather of the stacked batch of step t.
// Slot b of agent i takes word b & 3 of block b >> 2 of the agent's stream 0 at
// step t and maps it to a row of the agent's buffer; element e = b * row + c of
// the batch copies column c of that row.  Shared by the stand-alone gather
// kernel and by the prefetch role of the weight-gradient kernel.
#pragma once
#include "pop_dev.h"
#include "rng.h"

namespace pop {

// Floats of the stacked batch one thread copies.  Each workgroup waits for a trip to random rows and is the tail of a launch, so there
// should be no more of them than CUs, with as many loads in flight each as that takes.  Critics' tile launch of 256 agents at 42 floats per row, of 32 at
// 771 (us): every float's row drawn by its own thread, 4 and 13 floats per thread 275 and 115; rows drawn first, three workgroups per CU 261 and 101.
// us/step, three per CU / one: 80 agents 333.7 / 331, 32 SAC agents 205.5 / 204.5.
__host__ __device__ inline int gather_floats_per_thread(const PopDev& d) {
  for (int e = 4; e < 32; e *= 2)
    if ((int64_t)d.P * ((d.B * d.row + 256 * e - 1) / (256 * e)) <= kCUs) return e;
  return 32;
}
__host__ __device__ inline int gather_blocks_per_agent(const PopDev& d) {
  const int per = 256 * gather_floats_per_thread(d);
  return (d.B * d.row + per - 1) / per;
}
constexpr int kGatherLds = 256;            // words of LDS: the drawn rows of a workgroup's part of the batch

// Workgroup `block` (of gather_blocks_per_agent) of one agent: thread `tid` copies the floats
// (block * E + k) * 256 + tid, k < E, of the agent's stacked batch.  The rows of that part are drawn first, a thread per row
// (drawn by every thread for each of its floats, a generator block and two integer divisions per float, the tail of the critics' tile launch
// was longer than the rows take to fetch).
template <int E>
__device__ __forceinline__ void gather_run(const PopDev& d, uint32_t t, int agent, int block, int tid, uint32_t* drawn) {
  const HpDev hp = d.hp[agent];
  const uint32_t count = d.count[agent];
  const int row = d.row, total = d.B * row, base = block * E * 256, last = (base + E * 256 < total ? base + E * 256 : total) - 1;
  const float* src = d.replay + (size_t)agent * d.capacity * row;
  float* dst = d.batch + ((size_t)(t & 1u) * d.P + agent) * total;
  const float inv = 1.0f / (float)row;
  // e / row for e < 256 row <= 2^24: the quotient is off by less than 2^-14, half a row is 2^-11 of one at least
  auto row_of = [&](int e) { return (int)(((float)e + 0.5f) * inv); };
  const int b0 = row_of(base), rows = row_of(last) - b0 + 1;                 // at most B = 256
  if (tid < rows) {
    const int b = b0 + tid;
    const U4 blk = philox4x32_10(hp.seed_lo, hp.seed_hi, (uint32_t)(b >> 2), t, kStreamIndex, 0u);
    const uint32_t idx = index_from_word(pick(blk, (uint32_t)b & 3u), count);
    drawn[tid] = idx;
    if (b * row >= base) d.idx[((size_t)(t & 1u) * d.P + agent) * d.B + b] = idx;
  }
  __syncthreads();
  float v[E];
  // all loads of a thread go out before the first store: the rows are random, every load a trip to HBM
  auto at = [&](int k) {
    const int e = base + k * 256 + tid, ec = e <= last ? e : last, b = row_of(ec);
    return src + (size_t)drawn[b - b0] * row + (ec - b * row);
  };
  if (d.rows_past) {
    int zero = 0;
    asm volatile("" : "+s"(zero));                   // (two branches of equal addresses become one with ordinary loads)
#pragma unroll
    for (int k = 0; k < E; ++k) v[k] = __builtin_nontemporal_load(at(k) + zero);
  } else {
#pragma unroll
    for (int k = 0; k < E; ++k) v[k] = *at(k);
  }
#pragma unroll
  for (int k = 0; k < E; ++k) {
    const int e = base + k * 256 + tid;
    if (e <= last) dst[e] = v[k];
  }
}
// lds: kGatherLds words
__device__ inline void gather_block(const PopDev& d, uint32_t t, int agent, int block, int tid, void* lds) {
  uint32_t* drawn = static_cast<uint32_t*>(lds);
  switch (gather_floats_per_thread(d)) {
    case 4: gather_run<4>(d, t, agent, block, tid, drawn); break;
    case 8: gather_run<8>(d, t, agent, block, tid, drawn); break;
    case 16: gather_run<16>(d, t, agent, block, tid, drawn); break;
    default: gather_run<32>(d, t, agent, block, tid, drawn);
  }
}

}  // namespace pop
