// Wavefront-level MFMA building blocks for the per-agent MLP layers.
//
// The dense contractions of the update step (App. C of the paper: y = x W + b per population member, and the matching
// backward products) on 32x32 tiles: first layers and weight gradients on v_mfma_f32_32x32x2_f32 (one instruction
// multiplies a 32x2 slice of A by a 2x32 slice of B into a 32x32 fp32 tile held as 16 registers per lane), wide first
// layers and the 256-deep products of 32- and 64-row chains on v_mfma_f32_32x32x16_bf16 from split operands (SplitProduct below).  (16-row chains:
// mfma_tiles16.h.)
//
// Operand layout of the fp32 instruction on a 64-lane wavefront:
//   A: lane l supplies A[row = l & 31][k = l >> 5]
//   B: lane l supplies B[k = l >> 5][col = l & 31]
//   D: register v of lane l is D[row = 8 (v >> 2) + 4 (l >> 5) + (v & 3)][col = l & 31]
//
// A workgroup is 8 / NT wavefronts; for a [R x 256] output each wavefront owns
// 32 NT columns for all R = 32 MT rows, i.e. MT x NT tiles.  NT = 2, four wavefronts:
// tile nt holds the columns of parity nt: lane l has columns 64 wave + 2 (l & 31) + nt
// (tile_col), two neighbours, which it loads and stores as one 8-byte access.  NT = 1, eight wavefronts: column
// 32 wave + (l & 31), 4-byte accesses.
// The left operand (activations) lives in LDS and is shared by the
// wavefronts; the right operand (weights) is read by each wavefront straight
// from global memory/L2 into registers, because every weight element is used
// by exactly one wavefront of the workgroup -- staging it in LDS would add
// traffic and barriers without any reuse.
//
// The contraction index may be visited in any order as long as both operands
// agree, so one lane fetches 4 consecutive k of the LDS operand with a single
// 16-byte read and uses them in 4 successive MFMAs (lanes 0-31 take k0..k0+3,
// lanes 32-63 take k0+4..k0+7).
#pragma once
#include <hip/hip_runtime.h>
#include "pop_dev.h"

namespace pop {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

__device__ inline f32x16 mfma32(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// fp32 products on the bf16 matrix pipe.  v_mfma_f32_32x32x2_f32 takes 64 cycles for 4096 FLOP,
// v_mfma_f32_32x32x16_bf16 32 cycles for 32768: sixteen times the rate.  An fp32 value is the sum of three bf16 values
// (8 significand bits each, 24 in all): h its upper half-word (cut off: rounding would turn the largest finite values
// into infinity), m = bf16(x - h), l = x - h - m, the differences exact.  Of the nine products of two such sums six are
// taken,
//   x y = hx hy + (hx my + mx hy + mx my + hx ly + lx hy) + rest,   |rest| < 2^-21 |x y|, 2^-25 in the mean,
// at 6 / 16 of the time of the fp32 instructions.  The large products and the five small ones are summed in
// accumulators of their own (low), added once at the end: the matrix pipe rounds the accumulator after every
// instruction, and in one accumulator the small products would pay that rounding five times as often.  Relative
// error of a 256-deep product against 64 bits (2-norm): 0.70e-7, fp32 instructions 2.04e-7 (ReLU outputs x Glorot
// weights); 0.70e-7 / 2.05e-7 (sparse gradients x weights); 0.58e-7 / 1.44e-7 (activations x gradients); 0.94e-7 /
// 2.48e-7 (all terms positive); 1.14e-7 / 2.80e-7 (magnitudes over e^+-4); summed in one accumulator 2.2e-7; with h
// rounded 0.67, 0.67, 0.55, 0.94, 1.12e-7.
// Infinities and NaN: x - h is NaN for them, and so is every small sum they enter, but hx hy is what the fp32
// instructions would give, and it dwarfs a finite small sum.  So a small sum that is not finite counts as the largest
// finite value instead (Acc::add_finite, one instruction per element: 0.2 % of a step with 80 agents, 0.5 % with 256).
// A large sum overflows only where the sum of the terms' magnitudes does.
// Small values: bf16 has the exponents of fp32, and the parts of a value below 2^-110 (8e-34) lose what lies below
// 2^-134.  A product's absolute error grows by 2^-134 (sum |x| + sum |y|) at most; with operands of 1e-31 nothing shows,
// of 1e-34 the error is 2.8e-7 where the fp32 instructions have 2.0e-7, of 1e-37 2.7e-4.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

struct Split8 {                            // eight consecutive contraction elements of one lane: high, middle and low parts
  bf16x8 t[3];
};

// One pair of elements (2 i, 2 i + 1): eleven vector instructions (the differences as two-term bf16 dot products would
// be seven, but those run on the matrix pipe: 78 cycles beside a matrix instruction instead of 42).
__device__ inline void split_pair(float a, float b, int i, Split8& s) {
  const auto put = [&](int q, uint32_t u) {
    const bf16x2 h = __builtin_bit_cast(bf16x2, u);
    s.t[q][2 * i] = h[0];
    s.t[q][2 * i + 1] = h[1];
  };
  const uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
  put(0, __builtin_amdgcn_perm(ub, ua, 0x07060302u));          // the upper halves of both words
  a -= __uint_as_float(ua & 0xffff0000u);
  b -= __uint_as_float(ub & 0xffff0000u);
  const uint32_t m = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
  put(1, m);
  a -= __uint_as_float(m << 16);
  b -= __uint_as_float(m & 0xffff0000u);
  put(2, __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2)));
}
__device__ inline void split8(const float (&x)[8], Split8& s) {
#pragma unroll
  for (int i = 0; i < 4; ++i) split_pair(x[2 * i], x[2 * i + 1], i, s);
}
__device__ inline void split8(const f32x4& lo, const f32x4& hi, Split8& s) {
  const float x[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  split8(x, s);
}

// the six products in the order they are issued: parts of the left and of the right operand
constexpr int kSplitTerms = 6;
constexpr int kTermX[kSplitTerms] = {2, 0, 1, 1, 0, 0}, kTermW[kSplitTerms] = {0, 2, 1, 0, 1, 0};

__device__ inline f32x16 mfma32_bf16(const bf16x8& a, const bf16x8& b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Global store of a result that another workgroup of the SAME launch reads (THROUGH): a
// device-scope atomic store, which is written through the XCD's L2 to memory instead of
// waiting there as a dirty line, so that the producer only has to see its own stores
// acknowledged before it signals, not have the whole L2 written back.
template <bool THROUGH>
__device__ inline void put(float* p, float v) {
  if (THROUGH) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *p = v;
}
template <bool THROUGH>
__device__ inline void put_word(uint32_t* p, uint32_t v) {
  if (THROUGH) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *p = v;
}
// the same for two neighbouring floats at an 8-byte aligned address (a lane's two columns, tile_col)
template <bool THROUGH>
__device__ inline void put2(float* p, float a, float b) {
  if (THROUGH) {
    const unsigned long long word = (unsigned long long)__float_as_uint(a) | ((unsigned long long)__float_as_uint(b) << 32);
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else {
    *reinterpret_cast<f32x2*>(p) = f32x2{a, b};
  }
}

// a lane's NT neighbouring columns
__device__ inline void store_cols(float* p, const float (&h)[2]) { *reinterpret_cast<f32x2*>(p) = f32x2{h[0], h[1]}; }
__device__ inline void store_cols(float* p, const float (&h)[1]) { *p = h[0]; }
template <bool THROUGH>
__device__ inline void put_cols(float* p, const float (&h)[2]) { put2<THROUGH>(p, h[0], h[1]); }
template <bool THROUGH>
__device__ inline void put_cols(float* p, const float (&h)[1]) { put<THROUGH>(p, h[0]); }

__device__ inline int acc_row(int v, int lane) { return 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3); }
// Column (of 256) that a lane holds of tile nt of its wavefront's two accumulator tiles: the lane's two columns
// are neighbours, so that a forward product fetches both weights of a row with one 8-byte load (half the load
// instructions, which is what the forward products were short of).
// NT = 1 (eight wavefronts of 32 columns): neighbouring lanes hold neighbouring columns.
template <int NT = 2>
__device__ inline int tile_col(int wave, int nt, int lane) {
  return NT == 2 ? 64 * wave + 2 * (lane & 31) + nt : 32 * wave + (lane & 31);
}
// a lane's values of its NT columns (neighbours) as one access
template <int NT> struct ColsOf { typedef f32x2 T; };
template <> struct ColsOf<1> { typedef float T; };
__device__ inline float col_of(const f32x2& v, int nt) { return v[nt]; }
__device__ inline float col_of(float v, int) { return v; }

// NT = 32-column tiles per wavefront: 2 in layer chains of four wavefronts, 1 in those of eight (a workgroup spans 256
// columns) and in the weight-gradient tiles (128 columns per workgroup).
template <int MT, int NT = 2>
struct Acc {
  f32x16 t[MT][NT];
  __device__ inline void zero() {
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
      for (int b = 0; b < NT; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) t[a][b][v] = 0.0f;
  }
  // plus o, NaN and infinities in it as the largest finite value (the small sums of split products, above)
  __device__ inline void add_finite(const Acc& o) {
    const float most = 0x1.fffffep127f;
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
      for (int b = 0; b < NT; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) t[a][b][v] += __builtin_amdgcn_fmed3f(o.t[a][b][v], -most, most);
  }
};

// A weight matrix of n floats as a buffer resource: a load takes its address from a scalar and one 32-bit offset per
// lane.  From per-lane pointers each stream of loads keeps a 64-bit address per lane and needs two vector instructions
// with a wait between them per four loads; with the resource 32-row forward products of two workgroups on a CU take 15,400
// cycles instead of 17,600.  Vector registers, pointers / resource: k_target of 64 rows 244 / 212, of 32 rows 256 with 2 spilled / 228,
// of 16 rows 186 / 164; spilled by k_step (32 rows) 44 / 40, by k_actor of 32 rows at two per CU 50 / 39; k_critic about the same.
// Loads whose lane offset lies at or beyond n give zero (n <= 0: all of them); a scalar offset is
// outside that check, so where rows beyond the matrix are asked for (first layers) the resource starts at the rows of the block.
typedef __amdgpu_buffer_rsrc_t WeightsRsrc;
__device__ inline WeightsRsrc weights_rsrc(const float* W, int n) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(W), 0, 4 * (n < 0 ? 0 : n), 0x00020000);
}
__device__ inline f32x2 rsrc_load2(WeightsRsrc r, uint32_t lane_bytes, int floats) {
  return __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(r, lane_bytes, 4 * floats, 0));
}
template <int NT>
__device__ inline typename ColsOf<NT>::T rsrc_load_cols(WeightsRsrc r, uint32_t lane_bytes, int floats) {
  if constexpr (NT == 2) return rsrc_load2(r, lane_bytes, floats);
  else return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, lane_bytes, 4 * floats, 0));
}
__device__ inline f32x4 rsrc_load4(WeightsRsrc r, uint32_t lane_bytes, int floats) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, lane_bytes, 4 * floats, 0));
}

// First-layer weights of one lane for the leading 32 rows of W (k = 8 i + 4 half + j),
// fetched ahead of time so that the product does not wait for memory; rows at or beyond K are zero.
template <int NT = 2>
struct SmallW {
  float w[4][NT][4];
  __device__ inline void load(const float* __restrict__ W, int K, int wave, int lane) {
    const uint32_t off = 4u * (uint32_t)(4 * (lane >> 5) * kH + tile_col<NT>(wave, 0, lane));
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const auto v = rsrc_load_cols<NT>(weights_rsrc(W + 8 * i * kH, (K - 8 * i) * kH), off + 4 * j * kH, 0);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) w[i][nt][j] = col_of(v, nt);
      }
  }
};

// acc[r][c] += sum_{k<K} X[r][k] W[k][c]   (forward product x W) for a small fan-in K.
//   X: LDS, row stride ldx, rows [0, 32 MT); columns >= K up to the next
//      multiple of 8 must hold finite values (they meet zero weights);
//   W: global, row-major [K][256]; `pre` holds its first 32 rows already.
template <int MT, int NT>
__device__ inline void gemm_xw_small(const float* __restrict__ Xl, int ldx, int K, const float* __restrict__ W,
                                     const SmallW<NT>& pre, int wave, int lane, Acc<MT, NT>& acc) {
  const int half = lane >> 5, l32 = lane & 31;
  const int K8 = (K + 7) & ~7;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (8 * i < K8) {
      f32x4 a[MT];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        a[mt] = *reinterpret_cast<const f32x4*>(&Xl[(32 * mt + l32) * ldx + 8 * i + 4 * half]);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) acc.t[mt][nt] = mfma32(a[mt][j], pre.w[i][nt][j], acc.t[mt][nt]);
    }
  }
  const float* wcol = W + tile_col<NT>(wave, 0, l32);
  for (int k0 = 32; k0 < K8; k0 += 8) {              // fan-in beyond 32: plain loop
    float b[NT][4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int k = k0 + 4 * half + j;
      const auto v = *reinterpret_cast<const typename ColsOf<NT>::T*>(wcol + (size_t)(k < K ? k : 0) * kH);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) b[nt][j] = k < K ? col_of(v, nt) : 0.0f;
    }
    f32x4 a[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      a[mt] = *reinterpret_cast<const f32x4*>(&Xl[(32 * mt + l32) * ldx + k0 + 4 * half]);
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc.t[mt][nt] = mfma32(a[mt][j], b[nt][j], acc.t[mt][nt]);
  }
}

// The same product for a fan-in of several hundred, on the bf16 pipe (SplitProduct's six products, above): blocks of 16,
// contraction index 16 i + 8 s + 4 half + j at element 4 s + j of a lane, both operands split in registers, four weight
// blocks in flight beyond the two that `pre` holds.  For the critic chains whose slabs lie over the input tile (32 rows, four wavefronts); all
// others split the tile once per workgroup (gemm_xw_slabs, below).  With 376 inputs the first layers are three fifths of a chain's
// matrix work, and the fp32 instructions take 1024 cycles per block of 32 rows and wavefront; the 12 bf16 instructions
// and the splits of 12 pairs per lane some 700.  20 TD3 agents, obs 376 / act 17: 308 -> 271 us/step; 32 SAC agents 513 -> 464.
// Error against 64 bits (2-norm; both emulated in numpy, normal inputs x Glorot weights), fp32 sums / here: 393 inputs 3.5e-7 /
// 0.9e-7, 140 inputs 2.1e-7 / 0.6e-7, 72 inputs 1.5e-7 / 0.5e-7; where a row has only four inputs that are not zero 4.0e-8 / 3.5e-8, two
// 3.1e-8 / 3.4e-8, one 2.5e-8 / 3.5e-8.  Inputs and weights below 2^-110 lose low parts, as in the hidden products (above).
// X: as above; columns of the tile beyond K hold zeros (load_input_wide), and a block that would reach past the tile's
// row reads its last four columns instead, where the weights are zero.
__device__ inline void gemm_xw_deep(const float* __restrict__ Xl, int ldx, int K, const float* __restrict__ W, const SmallW<2>& pre, int wave,
                                    int lane, Acc<1, 2>& acc) {
  constexpr int PF = 4;
  const int half = lane >> 5, l32 = lane & 31;
  const int nb = (K + 15) >> 4;
  uint32_t off = 4u * (uint32_t)(4 * half * kH + tile_col<2>(wave, 0, lane));
  Acc<1, 2> low;
  low.zero();
  float b[PF][2][8];
  auto request = [&](float (&dst)[2][8], int blk) {
    const WeightsRsrc Wr = weights_rsrc(W + 16 * blk * kH, (K - 16 * blk) * kH);      // rows at or beyond K are zero
    asm("" : "+v"(off));                              // or copies of it are kept for each block in flight
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const f32x2 v = rsrc_load2(Wr, off + 4 * (8 * (e >> 2) + (e & 3)) * kH, 0);
      dst[0][e] = v[0];
      dst[1][e] = v[1];
    }
  };
  f32x4 xn[2];                                       // the LDS operand runs one block ahead
  auto lds_block = [&](int i) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int c = 16 * i + 8 * s + 4 * half;
      xn[s] = *reinterpret_cast<const f32x4*>(&Xl[l32 * ldx + (c < ldx - 4 ? c : ldx - 4)]);
    }
  };
  // block i with weights w; the LDS operand of block i + 1 and the loads of next() go out ahead of the matrix work
  auto block = [&](const float (&w)[2][8], int i, auto next) {
    Split8 x, ws[2];
    split8(xn[0], xn[1], x);
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) split8(w[nt], ws[nt]);
    lds_block(i + 1);
    next();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < kSplitTerms; ++q)
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) {
        f32x16& c = q == kSplitTerms - 1 ? acc.t[0][nt] : low.t[0][nt];
        c = mfma32_bf16(x.t[kTermX[q]], ws[nt].t[kTermW[q]], c);
      }
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int s = 0; s < PF; ++s) request(b[s], 2 + s);
  lds_block(0);
#pragma unroll
  for (int i = 0; i < 2; ++i)
    if (i < nb) {
      float w[2][8];
#pragma unroll
      for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int e = 0; e < 8; ++e) w[nt][e] = pre.w[2 * i + (e >> 2)][nt][e & 3];
      block(w, i, [] {});
    }
  int blk = 2;
  for (; blk + PF <= nb; blk += PF) {                // whole groups: no branch inside
#pragma unroll
    for (int s = 0; s < PF; ++s) block(b[s], blk + s, [&] { request(b[s], blk + s + PF); });
  }
#pragma unroll
  for (int s = 0; s < PF; ++s)
    if (blk + s < nb) block(b[s], blk + s, [] {});
  acc.add_finite(low);
}

// 256-deep contraction of 32 rows of an LDS operand with 32 columns per wavefront of a global operand Z (row-major
// [..][256]) on the fp32 instructions, for the weight-gradient tiles:  acc[r][c] += sum_k X[r][k] Z[k][c].  The
// contraction index is walked in blocks of 16.
struct ZBlock {                            // what one lane needs of Z for a block
  float w[8];                              // [4 s + j]  <->  index 16 i + 8 s + 4 half + j
  static constexpr int kPieces = 8;        // load instructions per block
  __device__ static inline const float* lane_base(const float* __restrict__ Z, int wave, int lane) {
    return Z + 4 * (lane >> 5) * kH + 32 * wave + (lane & 31);
  }
  __device__ inline void load_piece(const float* __restrict__ blk, int p) { w[p] = blk[(8 * (p >> 2) + (p & 3)) * kH]; }
  __device__ inline void load(const float* __restrict__ Z, int i, int wave, int lane) {
    const float* blk = lane_base(Z, wave, lane) + 16 * i * kH;
#pragma unroll
    for (int p = 0; p < kPieces; ++p) load_piece(blk, p);
  }
};

struct LdsBlock {                          // the LDS operand of one block
  f32x4 a[2];
  __device__ inline void load_piece(const float* __restrict__ Xl, int ldx, int k0, int lane, int s) {
    a[s] = *reinterpret_cast<const f32x4*>(&Xl[(lane & 31) * ldx + k0 + 8 * s + 4 * (lane >> 5)]);
  }
  __device__ inline void load(const float* __restrict__ Xl, int ldx, int k0, int lane) {
#pragma unroll
    for (int s = 0; s < 2; ++s) load_piece(Xl, ldx, k0, lane, s);
  }
};

// The MFMAs of one block with the loads of a later block (`nz` <- the block at `blk` when FEED, LDS operand `nx` <- columns
// nk0.. when FEEDX) dealt out between them, one piece behind an MFMA until they are used up (scheduling groups tell the
// compiler that order).  A matrix instruction keeps its pipe busy for 64 cycles after it issues; load instructions issued in
// that shadow cost nothing, while a whole block's worth of them between two blocks -- some 16 cycles each -- leaves
// the pipe idle for as long as they take to issue, where the other wavefront of the SIMD is no further along.
template <bool FEED, bool FEEDX>
__device__ inline void mfma_block_fed(const LdsBlock& x, const ZBlock& b, Acc<1, 1>& acc, ZBlock& nz, const float* __restrict__ blk,
                                      LdsBlock& nx, const float* __restrict__ Xl, int ldx, int nk0, int lane) {
  constexpr int M = 8, L = ZBlock::kPieces, LX = 2;
  if (FEEDX) nx.load(Xl, ldx, nk0, lane);
  if (FEED) {
#pragma unroll
    for (int p = 0; p < L; ++p) nz.load_piece(blk, p);
  }
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc.t[0][0] = mfma32(x.a[s][j], b.w[4 * s + j], acc.t[0][0]);
#pragma unroll
  for (int m = 0; m < M; ++m) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    if (FEEDX && m < LX) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    if (FEED && m < L) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
  }
  __builtin_amdgcn_sched_barrier(0);
}

// Fully unrolled with NB rotating buffers (block i + NB - 1 is requested under the MFMAs of block i): Z comes from memory
// rather than L2 and a block is only 512 cycles of matrix work.  z0: block 0, from the caller, who requests it as early as it
// can.  KB: blocks to contract over (16: all 256; 8: the half that Xl and Z point at).
template <int NB, int KB = 16>
__device__ inline void gemm256_unrolled(const float* __restrict__ Xl, int ldx, const float* __restrict__ Z, const ZBlock& z0,
                                        int wave, int lane, Acc<1, 1>& acc) {
  ZBlock zb[NB];
  LdsBlock xb[2];
  zb[0] = z0;
#pragma unroll
  for (int i = 1; i < NB - 1; ++i) zb[i].load(Z, i, wave, lane);
  xb[0].load(Xl, ldx, 0, lane);
  const float* zl = ZBlock::lane_base(Z, wave, lane);
  constexpr int step = 16 * kH;
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < KB; ++i) {
    const int n = i + NB - 1;
    if (n < KB) mfma_block_fed<true, true>(xb[i & 1], zb[i % NB], acc, zb[n % NB], zl + n * step, xb[(i + 1) & 1], Xl, ldx, 16 * (i + 1), lane);
    else if (i + 1 < KB) mfma_block_fed<false, true>(xb[i & 1], zb[i % NB], acc, zb[n % NB], zl, xb[(i + 1) & 1], Xl, ldx, 16 * (i + 1), lane);
    else mfma_block_fed<false, false>(xb[i & 1], zb[i % NB], acc, zb[n % NB], zl, xb[(i + 1) & 1], Xl, ldx, 0, lane);
  }
}

// The same product where Z is a critic's dZ2[b][c] = (bit (b, c) of the pattern) ? dq[b] w3[c] : 0, rebuilt from its factors
// (bit for bit what the chain multiplied): three vector instructions per element in the shadow of a 64-cycle matrix
// instruction instead of a 4-byte load, 128 KB less for a tile to fetch and 256 KB per network less to write and read.
// us/step with dZ2 in memory / rebuilt: 256 agents 1075 / 1034, 80 agents 346 / 338, shared critics 322 / 313, 10 agents
// 75.9 / 74.3; with a single agent the product of a tile takes 0.2 us longer (60.1 / 60.2).
template <int KB>
struct Dz2Factors {                        // for this lane's column
  static constexpr int kWords = KB / 2;
  uint32_t rows[kWords];                   // pattern of 32 batch rows each; shifted right by the lane's 4 (lane >> 5)
  float w3;
  // mask: [rows / 32][256] words from the first row on, at the tile's first column of this wavefront
  __device__ inline void load(const uint32_t* __restrict__ mask, const float* __restrict__ w, int lane) {
#pragma unroll
    for (int q = 0; q < kWords; ++q) rows[q] = mask[q * kH + (lane & 31)];
    w3 = w[lane & 31];
  }
};
template <int KB>
__device__ inline void gemm256_dz2(const float* __restrict__ Xl, int ldx, const float* __restrict__ dql, const Dz2Factors<KB>& f,
                                   int lane, Acc<1, 1>& acc) {
  const float* dqh = dql + 4 * (lane >> 5);
  LdsBlock xb[2];
  f32x4 dq[2];
  float z[2][8];
  auto request = [&](int i) {
    xb[i & 1].load(Xl, ldx, 16 * i, lane);
#pragma unroll
    for (int s = 0; s < 2; ++s) dq[s] = *reinterpret_cast<const f32x4*>(dqh + 16 * i + 8 * s);
  };
  auto rebuild = [&](int i) {
    const int rows = (int)(f.rows[i >> 1] >> (4 * (lane >> 5)));
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int keep = __builtin_amdgcn_sbfe(rows, 16 * (i & 1) + 8 * (e >> 2) + (e & 3), 1);
      z[i & 1][e] = __int_as_float(keep & __float_as_int(dq[e >> 2][e & 3] * f.w3));
    }
  };
  request(0);
  rebuild(0);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < KB; ++i) {                     // block i + 1 is read and rebuilt under the matrix instructions of block i
    if (i + 1 < KB) { request(i + 1); rebuild(i + 1); }
#pragma unroll
    for (int e = 0; e < 8; ++e) acc.t[0][0] = mfma32(xb[i & 1].a[e >> 2][e & 3], z[i & 1][e], acc.t[0][0]);
    if (i + 1 < KB) {
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if (m == 0) __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
        if (m > 3) __builtin_amdgcn_sched_group_barrier(0x002, 7, 0);   // the LDS has answered by then
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

template <int N> struct IntC { static constexpr int value = N; };
struct NoTail { __device__ inline void operator()() const {} };

// ---------------------------------------------------------------------------------------------
// 256-deep product of an LDS operand (fp32 tile, row stride kLda) with a global weight operand on the bf16 pipe:
//   forward  (TRANSPOSED = false): acc[r][c] += sum_k X[r][k] W[k][c], c in this wave's 32 NT columns
//   backward (TRANSPOSED = true):  acc[r][k] += sum_n Z[r][n] W[k][n], k in this wave's 32 NT columns
// W is a [256][256] hidden matrix in the order of w2_index<PLAIN> in both cases.  Matrix and vector instructions share the issue port (measured: about five
// cycles for either beside the other; a matrix instruction keeps its pipe for 32), and a pair of elements costs eleven
// vector instructions to split, so the number of splits decides: a weight is used by one wavefront and split in its
// registers, once per 32 MT rows; the LDS operand is used by all wavefronts and split once per workgroup, 64
// columns (a slab) at a time, into three bf16 planes in LDS from which the wavefronts read their operands ready for
// use.  Per wavefront and 16-deep block: 6 MT NT matrix instructions, 44 NT + 11 MT NT / 2 vector instructions (44 NT + 44 MT where
// every wavefront splits both operands itself).
// 64 rows on one CU, us per product with the weights in L2: two 32-row workgroups on the fp32 instructions 16.9; here
// 10.9 forward and 14.2 backward as two 32-row workgroups, 8.9 and 8.4 as one of 64 rows (zero weights; 13.3, 15.2,
// 11.2, 10.9 with random ones, under which the clock falls from 2.3 to 1.9 GHz).  With both operands split in registers
// 11.4, 14.6, 9.7, 8.9.  Differences by two-term bf16 dot products instead of shift and subtract: slower than fp32 (they run on the matrix pipe).

// The weights one lane needs for a 16-deep block i = 2 D + o: contraction indices 32 D + 16 half + 8 o + e, e < 8.  Two
// blocks cover whole 128-byte lines of the transposed operand (a lane reads 64 bytes of one row of W).
template <bool TRANSPOSED, int NT = 2, bool PLAIN = false>
struct WeightRaw {
  __device__ static constexpr int at(int k, int n) { return w2_index<PLAIN>(k, n); }
  float w[NT][8];                           // [column tile][e]
  static constexpr int kPieces = TRANSPOSED ? 2 * NT : 8;           // load instructions per block
  static constexpr int kGroup = TRANSPOSED ? w2_index<PLAIN>(0, 64) : w2_index<PLAIN>(64, 0);   // floats from one group of four blocks to the next
  __device__ static constexpr int offset(int i) {
    const int k = 32 * (i >> 1) + 8 * (i & 1);
    return TRANSPOSED ? at(0, k) : at(k, 0);
  }
  __device__ static inline WeightsRsrc rsrc(const float* W) { return weights_rsrc(W, kH * kH); }
  __device__ static inline uint32_t lane_bytes(int wave, int lane) {
    const int half = lane >> 5, col = tile_col<NT>(wave, 0, lane);
    return 4u * (uint32_t)(TRANSPOSED ? at(col, 16 * half) : at(16 * half, col));
  }
  __device__ inline void load_piece(WeightsRsrc W, uint32_t lane_off, int blk, int p) {
    if (TRANSPOSED) {
      const int nt = p >> 1, s = p & 1;              // two columns are neighbouring rows of W, the first one even
      const f32x4 v = rsrc_load4(W, lane_off + 4 * at(nt, 4 * s), blk);
#pragma unroll
      for (int j = 0; j < 4; ++j) w[nt][4 * s + j] = v[j];
    } else {
      const auto v = rsrc_load_cols<NT>(W, lane_off + 4 * at(p & 3, 0), blk + at(p & ~3, 0));
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) w[nt][p] = col_of(v, nt);
    }
  }
  __device__ inline void load_block(WeightsRsrc W, uint32_t lane_off, int blk) {
#pragma unroll
    for (int p = 0; p < kPieces; ++p) load_piece(W, lane_off, blk, p);
  }
  __device__ inline void load(const float* __restrict__ W, int i, int wave, int lane) {
    load_block(rsrc(W), lane_bytes(wave, lane), offset(i));
  }
};

// A slab: columns [64 s, 64 s + 64) of the LDS operand as three planes [32 MT][72] of bf16 (a row stride of 36 words:
// 16-byte accesses of neighbouring rows fall on different banks).  Two buffers.
constexpr int kSlabLd = 72;
template <int MT>
constexpr int slab_floats() { return 3 * 32 * MT * kSlabLd / 2; }
template <int MT, int NT>
struct SlabItem {                          // this thread's share of a slab: Q times E neighbours of a row
  static constexpr int E = MT * NT == 1 ? 4 : 8, Q = MT * NT == 4 ? 2 : 1, kPerRow = 64 / E;
  f32x4 x[Q][E / 4];
  __device__ inline void read(const float* __restrict__ Xl, int s, int tid, int q) {
    const float* p = Xl + (32 * q + tid / kPerRow) * kLda + 64 * s + E * (tid % kPerRow);
#pragma unroll
    for (int i = 0; i < E / 4; ++i) x[q][i] = *reinterpret_cast<const f32x4*>(p + 4 * i);
  }
  // of a tile with rows of ldx floats, the last four of which hold zeros: they stand in for what lies beyond
  __device__ inline void read_to(const float* __restrict__ Xl, int ldx, int s, int tid, int q) {
    const float* p = Xl + (32 * q + tid / kPerRow) * ldx;
    const int c = 64 * s + E * (tid % kPerRow);
#pragma unroll
    for (int i = 0; i < E / 4; ++i) x[q][i] = *reinterpret_cast<const f32x4*>(p + (c + 4 * i < ldx - 4 ? c + 4 * i : ldx - 4));
  }
  __device__ inline void put(float* __restrict__ slab, int tid, int q) const {
    Split8 v;
#pragma unroll
    for (int i = 0; i < E / 2; ++i) split_pair(x[q][i / 2][2 * (i & 1)], x[q][i / 2][2 * (i & 1) + 1], i, v);
    __bf16* b = reinterpret_cast<__bf16*>(slab) + (32 * q + tid / kPerRow) * kSlabLd + E * (tid % kPerRow);
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      if constexpr (E == 8) *reinterpret_cast<bf16x8*>(b + p * 32 * MT * kSlabLd) = v.t[p];
      else *reinterpret_cast<bf16x4*>(b + p * 32 * MT * kSlabLd) = __builtin_shufflevector(v.t[p], v.t[p], 0, 1, 2, 3);
    }
  }
};

// SLABS: as above; otherwise every wavefront splits the LDS operand itself, for chains whose scratch leaves no room for
// the slabs (SAC with 64 rows).
template <int MT, bool TRANSPOSED, bool SLABS, int NT, bool PLAIN>
struct SplitProduct {
  using Raw = WeightRaw<TRANSPOSED, NT, PLAIN>;
  static_assert(NT == 2 || SLABS, "eight wavefronts read the left operand from the slabs");
  Split8 x[2][MT], w[2];                   // the LDS operand of this block and the next, the weights of the two column tiles (NT = 1: of this block and the next)
  SlabItem<MT, NT> item;
  Acc<MT, NT> low;
  f32x4 xr[SLABS ? 1 : MT][2];             // the LDS operand as read, where there are no slabs

  // block b of the slab in this lane's layout
  __device__ inline void read_x(Split8 (&dst)[MT], const float* __restrict__ slab, int b, int lane) const {
    const __bf16* p = reinterpret_cast<const __bf16*>(slab) + (lane & 31) * kSlabLd + 32 * (b >> 1) + 16 * (lane >> 5) + 8 * (b & 1);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int q = 0; q < 3; ++q) dst[mt].t[q] = *reinterpret_cast<const bf16x8*>(p + (q * 32 * MT + 32 * mt) * kSlabLd);
  }
  __device__ inline void read_raw(const float* __restrict__ Xl, int i, int lane) {      // block i of the whole tile
#pragma unroll
    for (int mt = 0; mt < (SLABS ? 0 : MT); ++mt) {
      const float* p = Xl + (32 * mt + (lane & 31)) * kLda + 32 * (i >> 1) + 16 * (lane >> 5) + 8 * (i & 1);
      xr[mt][0] = *reinterpret_cast<const f32x4*>(p);
      xr[mt][1] = *reinterpret_cast<const f32x4*>(p + 4);
    }
  }
  __device__ inline void split_raw(Split8 (&dst)[MT]) const {
#pragma unroll
    for (int mt = 0; mt < (SLABS ? 0 : MT); ++mt) split8(xr[mt][0], xr[mt][1], dst[mt]);
  }
  __device__ inline void multiply(const Split8 (&xc)[MT], const Split8& wc, int nt, Acc<MT, NT>& acc) {
#pragma unroll
    for (int q = 0; q < kSplitTerms; ++q)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        f32x16& c = q == kSplitTerms - 1 ? acc.t[mt][nt] : low.t[mt][nt];
        c = mfma32_bf16(xc[mt].t[kTermX[q]], wc.t[kTermW[q]], c);
      }
  }
  // One block B (0 .. 3) of a group: the matrix instructions of column tile 0 with, dealt out between them, the split
  // of tile 1's weights and the reads of the next block's LDS operand (from `xs`, block (B + 1) & 3), then those of tile 1 with the
  // split of the next block's tile 0.  Beside them this thread's share of the next slab (SLAB: `nslab`): read in block 0,
  // split and written in blocks 1 and 2.  FEED: the weights four blocks on go into the registers of this
  // block -- transposed: of this and the block before, in odd blocks, so that both halves of a line are asked for together.
  template <int B, bool NEXT, bool SLAB, bool FEED>
  __device__ inline void block(Acc<MT, NT>& acc, Raw& wp, Raw& wc, const Raw& wn, WeightsRsrc W, uint32_t lane_off, int wg,
                               const float* __restrict__ xs, const float* __restrict__ Xl, int s, float* __restrict__ nslab,
                               int tid, int lane) {
    constexpr int M = kSplitTerms * MT, CUR = B & 1;
    constexpr bool stage = SLABS && SLAB, put = stage && B >= 1 && B <= SlabItem<MT, NT>::Q;
    constexpr int loads1 = !FEED ? 0 : TRANSPOSED ? (B & 1 ? 4 : 0) : 8;
    constexpr int loads = !FEED ? 0 : TRANSPOSED ? (B & 1 ? 8 : 0) : 8;
    asm("" : "+v"(lane_off));                         // or the constants added to it are hoisted into registers of their own
    if constexpr (NT == 1) {                          // one tile: all of it beside the matrix instructions of the block
      if (NEXT) { read_x(x[CUR ^ 1], xs, (B + 1) & 3, lane); split8(wn.w[0], w[CUR ^ 1]); }
      if (stage && B == 0) item.read(Xl, s + 1, tid, 0);
      if (put) item.put(nslab, tid, 0);
      if (FEED && TRANSPOSED && (B & 1)) { wp.load_block(W, lane_off, wg + Raw::offset(B + 3)); wc.load_block(W, lane_off, wg + Raw::offset(B + 4)); }
      if (FEED && !TRANSPOSED) wc.load_block(W, lane_off, wg + Raw::offset(B + 4));
      multiply(x[CUR], w[CUR], 0, acc);
#pragma unroll
      for (int m = 0; m < M; ++m) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if (NEXT) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        if (loads1 * m < 8 * M && loads1) __builtin_amdgcn_sched_group_barrier(0x020, (loads1 + M - 1) / M, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, ((NEXT ? 44 : 0) + (put ? 5 * SlabItem<MT, NT>::E + 4 : 0) + M - 1) / M + 1, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    } else {
    split8(wc.w[1], w[1]);
    if (NEXT && SLABS) read_x(x[CUR ^ 1], xs, (B + 1) & 3, lane);
    if (NEXT && !SLABS) read_raw(Xl, 4 * s + B + 1, lane);
    if (stage && B == 0) {
#pragma unroll
      for (int q = 0; q < SlabItem<MT, NT>::Q; ++q) item.read(Xl, s + 1, tid, q);
    }
    multiply(x[CUR], w[0], 0, acc);
#pragma unroll
    for (int m = 0; m < M; ++m) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (NEXT) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, (44 + M - 1) / M, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (NEXT) split8(wn.w[0], w[0]);
    if (NEXT && !SLABS) split_raw(x[CUR ^ 1]);
    if (put) item.put(nslab, tid, B - 1);
    if (FEED && TRANSPOSED && (B & 1)) { wp.load_block(W, lane_off, wg + Raw::offset(B + 3)); wc.load_block(W, lane_off, wg + Raw::offset(B + 4)); }
    if (FEED && !TRANSPOSED) wc.load_block(W, lane_off, wg + Raw::offset(B + 4));
    multiply(x[CUR], w[1], 1, acc);
#pragma unroll
    for (int m = 0; m < M; ++m) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (loads * m < 8 * M && loads) __builtin_amdgcn_sched_group_barrier(0x020, (loads + M - 1) / M, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, ((NEXT ? (SLABS ? 44 : 44 + 44 * MT) : 0) + (put ? 44 : 0) + M - 1) / M + 1, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    }
  }
  // Four blocks, slab s.  The barrier that completes the next slab stands before the last block, whose operand is in
  // registers by then: the first operand of the next slab arrives under it.
  template <bool LAST, class Tail>
  __device__ inline void group(Acc<MT, NT>& acc, Raw& b0, Raw& b1, Raw& b2, Raw& b3, WeightsRsrc W, uint32_t lane_off, int wg,
                               const float* __restrict__ Xl, int s, float* __restrict__ cur, float* __restrict__ nxt, int tid, int lane, Tail& tail) {
    block<0, true, !LAST, !LAST>(acc, b3, b0, b1, W, lane_off, wg, cur, Xl, s, nxt, tid, lane);
    block<1, true, !LAST, !LAST>(acc, b0, b1, b2, W, lane_off, wg, cur, Xl, s, nxt, tid, lane);
    if (LAST) tail();
    block<2, true, !LAST, !LAST>(acc, b1, b2, b3, W, lane_off, wg, cur, Xl, s, nxt, tid, lane);
    if (!LAST && SLABS) __syncthreads();
    block<3, !LAST, false, !LAST>(acc, b2, b3, b0, W, lane_off, wg, nxt, Xl, s, nxt, tid, lane);
  }
  // b0: block 0, from the caller, who requests it as early as it can (typically under the previous product); tail() runs
  // once no further weight block is needed, so that the caller can start the loads of the next layer under the last
  // two blocks.  slabs: 2 slab_floats<MT>() floats of LDS.  With slabs, every wavefront
  // has read the tile when any returns.
  template <class Tail>
  __device__ inline void run(const float* __restrict__ Xl, const float* __restrict__ W, Raw& b0, float* __restrict__ slabs, int wave, int lane,
                             Acc<MT, NT>& acc, Tail& tail) {
    const int tid = 64 * wave + lane;
    float* s0 = slabs;
    float* s1 = slabs + slab_floats<MT>();
    Raw b1, b2, b3;
    if (SLABS) {
#pragma unroll
      for (int q = 0; q < SlabItem<MT, NT>::Q; ++q) item.read(Xl, 0, tid, q);
    } else {
      read_raw(Xl, 0, lane);
    }
    b1.load(W, 1, wave, lane);
    b2.load(W, 2, wave, lane);
    b3.load(W, 3, wave, lane);
    low.zero();
    POP_MARK(20);
    const WeightsRsrc Wr = Raw::rsrc(W);
    const uint32_t lane_off = Raw::lane_bytes(wave, lane);
    int wg = 0;                                      // floats to the group
    if (SLABS) {
#pragma unroll
      for (int q = 0; q < SlabItem<MT, NT>::Q; ++q) item.put(s0, tid, q);
      __syncthreads();
      read_x(x[0], s0, 0, lane);
    } else {
      split_raw(x[0]);
    }
    split8(b0.w[0], w[0]);
    __builtin_amdgcn_sched_barrier(0);
    // (Left as a loop, the compiler moves the head of the last group into it for eight wavefronts' forward products and copies
    // the accumulators: 38 registers spilled by the product alone.)
    const auto slab = [&](int s) {
      group<false>(acc, b0, b1, b2, b3, Wr, lane_off, wg, Xl, s, s0, s1, tid, lane, tail);
      wg += Raw::kGroup;
      float* q = s0; s0 = s1; s1 = q;
    };
    if constexpr (NT == 1 && !TRANSPOSED) {
#pragma unroll
      for (int s = 0; s < 3; ++s) slab(s);
    } else {
#pragma unroll 1
      for (int s = 0; s < 3; ++s) slab(s);
    }
    group<true>(acc, b0, b1, b2, b3, Wr, lane_off, wg, Xl, 3, s0, s1, tid, lane, tail);
    acc.add_finite(low);
    POP_MARK(24);
  }
};

// gemm_xw_deep's product (the same instructions in the same order, so the same bits) with the input tile split once per
// workgroup, a slab of 64 columns at a time, instead of by every wavefront: per wavefront and block of 16 rows of W 44 NT + 11 vector
// instructions beside 6 NT matrix instructions (32 rows), where there were 44 NT + 44.  Four weight blocks in registers, the two of `pre` the first;
// blocks beyond K (a request ahead) read as zero.  slabs: as for gemm256, idle when the function is called and, after the next barrier, again.
template <int MT, int NT>
__device__ inline void gemm_xw_slabs(const float* __restrict__ Xl, int ldx, int K, const float* __restrict__ W,
                                     const SmallW<NT>& pre, float* __restrict__ slabs, int wave, int lane, Acc<MT, NT>& acc) {
  using Item = SlabItem<MT, NT>;
  const int half = lane >> 5, l32 = lane & 31, tid = 64 * wave + lane;
  const int nb = (K + 15) >> 4;
  uint32_t off = 4u * (uint32_t)(4 * half * kH + tile_col<NT>(wave, 0, lane));
  Acc<MT, NT> low;
  low.zero();
  float b[4][NT][8];
  auto request = [&](float (&dst)[NT][8], int blk) {
    const WeightsRsrc Wr = weights_rsrc(W + 16 * blk * kH, (K - 16 * blk) * kH);      // rows at or beyond K are zero
    asm("" : "+v"(off));                              // or copies of it are kept for each block in flight
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const auto v = rsrc_load_cols<NT>(Wr, off + 4 * (8 * (e >> 2) + (e & 3)) * kH, 0);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) dst[nt][e] = col_of(v, nt);
    }
  };
  Item item;
  float* cur = slabs;
  float* nxt = slabs + slab_floats<MT>();
  Split8 x[2][MT];
  auto read_x = [&](Split8 (&dst)[MT], const float* slab, int blk) {                  // columns 16 blk + 8 s + 4 half of the slab
    const __bf16* p = reinterpret_cast<const __bf16*>(slab) + l32 * kSlabLd + 16 * blk + 4 * half;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const __bf16* r = p + (q * 32 * MT + 32 * mt) * kSlabLd;
        const bf16x4 lo = *reinterpret_cast<const bf16x4*>(r), hi = *reinterpret_cast<const bf16x4*>(r + 8);
        dst[mt].t[q] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      }
  };
  // block B of the slab; FULL: the slab has four and this thread's share of the next one is staged beside them
  auto block = [&](auto B_, auto FULL_, int s, bool next) {
    constexpr int B = decltype(B_)::value;
    constexpr bool FULL = decltype(FULL_)::value, stage = FULL && B == 0, put = FULL && B >= 1 && B <= Item::Q;
    constexpr int M = kSplitTerms * MT * NT;
    Split8 ws[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) split8(b[B][nt], ws[nt]);
    request(b[B], 4 * s + B + 4);
    if (FULL && B == 3) __syncthreads();             // the next slab is complete
    if (next) read_x(x[(B + 1) & 1], B == 3 ? nxt : cur, (B + 1) & 3);
    if (stage) {
#pragma unroll
      for (int q = 0; q < Item::Q; ++q) item.read_to(Xl, ldx, s + 1, tid, q);
    }
    if (put) item.put(nxt, tid, B - 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < kSplitTerms; ++q)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          f32x16& c = q == kSplitTerms - 1 ? acc.t[mt][nt] : low.t[mt][nt];
          c = mfma32_bf16(x[B & 1][mt].t[kTermX[q]], ws[nt].t[kTermW[q]], c);
        }
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int e = 0; e < 8; ++e) b[i][nt][e] = pre.w[2 * i + (e >> 2)][nt][e & 3];
  request(b[2], 2);
  request(b[3], 3);
#pragma unroll
  for (int q = 0; q < Item::Q; ++q) item.read_to(Xl, ldx, 0, tid, q);
#pragma unroll
  for (int q = 0; q < Item::Q; ++q) item.put(cur, tid, q);
  __syncthreads();
  read_x(x[0], cur, 0);
  int s = 0;
#pragma unroll 1
  for (; 4 * s + 4 <= nb; ++s) {                     // whole slabs: no branch inside
    block(IntC<0>(), IntC<1>(), s, true);
    block(IntC<1>(), IntC<1>(), s, true);
    block(IntC<2>(), IntC<1>(), s, true);
    block(IntC<3>(), IntC<1>(), s, true);
    float* q = cur; cur = nxt; nxt = q;
  }
  const int rem = nb - 4 * s;
  if (rem > 0) block(IntC<0>(), IntC<0>(), s, rem > 1);
  if (rem > 1) block(IntC<1>(), IntC<0>(), s, rem > 2);
  if (rem > 2) block(IntC<2>(), IntC<0>(), s, false);
  acc.add_finite(low);
}

template <int MT, bool TRANSPOSED, bool SLABS, int NT, bool PLAIN, class Tail>
__device__ inline void gemm256(const float* __restrict__ Xl, const float* __restrict__ W, WeightRaw<TRANSPOSED, NT, PLAIN>& b0,
                               float* __restrict__ slabs, int wave, int lane, Acc<MT, NT>& acc, Tail tail) {
  SplitProduct<MT, TRANSPOSED, SLABS, NT, PLAIN> p;
  p.run(Xl, W, b0, slabs, wave, lane, acc, tail);
  if (!SLABS) __syncthreads();                       // every wavefront has read the tile
}

// ReLU epilogue of a hidden layer: Y = max(acc + b, 0) goes to LDS (row stride
// kLda) and, when Yg != nullptr, to global memory as [rows][256].  Returns the
// activation pattern of this lane's elements (bb = the bias values of
// this lane's NT columns, tile_col, loaded by the caller ahead of the product), bit (NT mt + nt) 16 + v, so that
// the backward pass can apply ReLU' without re-reading the activations: the
// input-gradient product leaves element (row, col) in the same lane and
// register as the forward product did.
template <int MT, bool THROUGH = false, int NT = 2>
__device__ inline uint64_t relu_store(const Acc<MT, NT>& acc, const float (&bb)[NT], float* __restrict__ Yl,
                                      float* __restrict__ Yg, int wave, int lane) {
  uint64_t mask = 0;
  const int col = tile_col<NT>(wave, 0, lane);       // two columns of a lane go out as one 8-byte store
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int row = 32 * mt + acc_row(v, lane);
      float h[NT];
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        h[nt] = fmaxf(acc.t[mt][nt][v] + bb[nt], 0.0f);
        if (h[nt] > 0.0f) mask |= 1ull << ((NT * mt + nt) * 16 + v);
      }
      store_cols(&Yl[row * kLda + col], h);
      if (Yg) put_cols<THROUGH>(Yg + (size_t)row * kH + col, h);
    }
  return mask;
}

template <int NT = 2>
__device__ inline bool mask_bit(uint64_t mask, int mt, int nt, int v) {
  return (mask >> ((NT * mt + nt) * 16 + v)) & 1ull;
}

// Thin products on the vector ALU (heads with 1..8 outputs, action gradient):
// out[r*stride + j] = sum_{c<256} X[r][c] V[j*256 + c],  r < R, j < J <= 8, X and V in LDS.
// Thread t works on rows (t >> 3) + 32 i with column groups 32 q + 4 (t & 7);
// 8 neighbouring lanes share a row and are summed with lane shuffles.
// `stride`: row stride of `outl` (kMaxAct unless the caller keeps wider rows).
// THREADS / 8 rows at a time.
template <int R, int THREADS = kThreads>
__device__ inline void thin_dot(const float* __restrict__ Xl, const float* __restrict__ V, int J,
                                float* __restrict__ outl, int tid, int stride = kMaxAct) {
  const int p = tid & 7;
  for (int i = 0; i < (8 * R + THREADS - 1) / THREADS; ++i) {
    if (8 * R < THREADS && tid >= 8 * R) break;
    const int r = (tid >> 3) + THREADS / 8 * i;
    float s[kMaxAct];
#pragma unroll
    for (int j = 0; j < kMaxAct; ++j) s[j] = 0.0f;
#pragma unroll 2
    for (int q = 0; q < 8; ++q) {
      const int c = 32 * q + 4 * p;
      const f32x4 x = *reinterpret_cast<const f32x4*>(&Xl[r * kLda + c]);
#pragma unroll
      for (int j = 0; j < kMaxAct; ++j) {
        if (j < J) {
          const f32x4 w = *reinterpret_cast<const f32x4*>(&V[j * kH + c]);
          s[j] += x[0] * w[0] + x[1] * w[1] + x[2] * w[2] + x[3] * w[3];
        }
      }
    }
#pragma unroll
    for (int j = 0; j < kMaxAct; ++j) {
      if (j < J) {
        float v = s[j];
        v += __shfl_xor(v, 1);
        v += __shfl_xor(v, 2);
        v += __shfl_xor(v, 4);
        if (p == 0) outl[r * stride + j] = v;
      }
    }
  }
}

}  // namespace pop
