// float32 products on the 16-bit matrix cores (gfx950).
//
// Three bf16 parts.  A float32 number is the exact sum of three bf16 numbers:
// the top eight significand bits (cut off, so nothing overflows), the next
// eight (rounded) and the rest, which fits in eight.  Of the nine products of
// two such sums the six largest are accumulated in float32; the three left out
// are below 2^-23 of the product and of either sign.
//
// Two f16 parts, where the operands' magnitudes are known.  Scaled by a power
// of two so that the largest magnitude lies in [2^14, 2^15), a float32 number
// is the sum of two f16 numbers up to 2^-23 of itself (2^-40 of the largest,
// where that is more); three products are accumulated, and the one left out
// is below 2^-22 of the product.
//
// The two forms are published: G. Henry, P. Tang and A. Heinecke, "Leveraging
// the bfloat16 artificial intelligence datatype for higher-precision
// computations", ARITH 2019 (three bf16 parts); H. Ootomo and R. Yokota,
// "Recovering single precision accuracy from Tensor Cores while surpassing the
// FP32 theoretical peak performance", 2022 (two scaled half-precision parts).
//
// The rounding of the float32 accumulators dominates the errors.  A product
// of parts rounds its sum once per 16 terms, a float32 MFMA once per 4 (16x16x4)
// or 2 (32x32x2).  Where all six products of three parts round one sum, runs
// of 512 terms are 1.52 times as far from float64 as a float32 sum rounded
// once per 4 terms; with the small products in a set of sums of their own
// (SplitAcc) 0.59 times.  One sum for the three products of two parts rounds
// less than half as often as the 32x32x2 form that it replaces (dot products
// of 512 / 2048 / 18816 terms, relative 2-norm: 2.6e-7 / 5e-7 / 1.9e-6 against
// 4.0e-7 / 7.7e-7 / 2.4e-6).
//
// The matrix cores sustain 145 TFLOP/s in float32 and 1850 in bf16 and f16 on
// random operands, so six products take 0.47 of the time and three 0.24; and
// vector instructions (the splitting) issue beside these MFMAs, while they
// stall float32 ones.
// An infinite operand gives NaN here (one of its parts is NaN, and infinity
// times a zero part): the kernels take such sums again in float32.
#pragma once

#include "internal.h"

namespace hav {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Exponent e such that a magnitude m (the bits of a nonnegative float) scaled
// by 2^e lies in [2^14, 2^15) (below it for subnormals and zero).
__host__ __device__ inline int split_exp(uint32_t bits) { return 141 - (int)(bits >> 23); }
constexpr int kNonFiniteExp = 141 - 255;  // of an infinite or NaN magnitude

// The NPART parts of two floats, each part's pair packed (low half: a).
template <int NPART>
struct Split2 {
  uint32_t p[NPART];
};
template <int NPART>
__device__ inline Split2<NPART> split2(float a, float b) {
  Split2<NPART> s;
  if constexpr (NPART == 3) {
    const uint32_t ua = __builtin_bit_cast(uint32_t, a), ub = __builtin_bit_cast(uint32_t, b);
    auto pk = [](float x, float y) {
      return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){x, y}, bf16x2));
    };
    s.p[0] = __builtin_amdgcn_perm(ub, ua, 0x07060302u);  // the upper halves of a, b
    const float ra = a - __builtin_bit_cast(float, ua & 0xffff0000u);
    const float rb = b - __builtin_bit_cast(float, ub & 0xffff0000u);
    s.p[1] = pk(ra, rb);
    s.p[2] = pk(ra - __builtin_bit_cast(float, s.p[1] << 16), rb - __builtin_bit_cast(float, s.p[1] & 0xffff0000u));
  } else {
    const f16x2 h = __builtin_convertvector((f32x2){a, b}, f16x2);
    const f16x2 l = __builtin_convertvector((f32x2){a - (float)h.x, b - (float)h.y}, f16x2);
    s.p[0] = __builtin_bit_cast(uint32_t, h);
    s.p[1] = __builtin_bit_cast(uint32_t, l);
  }
  return s;
}

template <int NPART>
__device__ inline f32x16 mfma_part(u32x4 a, u32x4 b, f32x16 c) {
  if constexpr (NPART == 3)
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                   0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0,
                                                  0);
}
// The products taken, small ones first: parts (of a, of b).
template <int NPART>
struct SplitOrder;
template <>
struct SplitOrder<3> {
  static constexpr int n = 6, a[6] = {2, 0, 1, 1, 0, 0}, b[6] = {0, 2, 1, 0, 1, 0};
};
template <>
struct SplitOrder<2> {
  static constexpr int n = 3, a[3] = {1, 0, 0}, b[3] = {0, 1, 0};
};

// Operand tiles in LDS for 32x32x16 MFMAs: a stage holds 16 k of ROWS rows as
// NPART planes (the parts), each two halves of 8 k, each half ROWS pieces of
// 16 bytes (a row's 8 k).  Lane (l, h) of a wave reads row l's piece of half
// h: 16 consecutive lanes read 256 consecutive bytes.  A half is followed by
// 128 bytes, so that the two halves of a row fall into different banks for
// 8-byte writes of four lanes per row.
template <int ROWS, int NPART>
struct SplitTile {
  static constexpr int kHalf = ROWS * 16 + 128;
  static constexpr int kPlane = 2 * kHalf;
  static constexpr int kBytes = NPART * kPlane;
  // Four consecutive k (piece q of 4) of a row.
  __device__ static void put4(char* tile, int row, int q, f32x4 v) {
    const Split2<NPART> a = split2<NPART>(v.x, v.y), b = split2<NPART>(v.z, v.w);
    char* d = tile + (q >> 1) * kHalf + row * 16 + (q & 1) * 8;
#pragma unroll
    for (int i = 0; i < NPART; ++i) *(u32x2*)(d + i * kPlane) = u32x2{a.p[i], b.p[i]};
  }
  // Eight consecutive k (half h) of a row.
  __device__ static void put8(char* tile, int row, int h, const float* v) {
    Split2<NPART> s[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) s[i] = split2<NPART>(v[2 * i], v[2 * i + 1]);
    char* d = tile + h * kHalf + row * 16;
#pragma unroll
    for (int i = 0; i < NPART; ++i)
      *(u32x4*)(d + i * kPlane) = u32x4{s[0].p[i], s[1].p[i], s[2].p[i], s[3].p[i]};
  }
  __device__ static u32x4 get(const char* tile, int plane, int row, int h) {
    return *(const u32x4*)(tile + plane * kPlane + h * kHalf + row * 16);
  }
};

// The float32 sums of a wave's MI x NI blocks of 32 x 32.  DUAL: the products
// of the largest parts are summed by themselves, so that the full sum rounds
// once per 16 terms, and the small ones (2^-8 of them and less) in a second
// set, added at the end; without it every product rounds the one sum.
template <int MI, int NI, bool DUAL>
struct SplitAcc {
  f32x16 sum[MI][NI];
  f32x16 low[DUAL ? MI : 1][DUAL ? NI : 1];
  __device__ void clear() {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          sum[i][j][r] = 0.0f;
          if constexpr (DUAL) low[i][j][r] = 0.0f;
        }
  }
  // Adds product q (SplitOrder) of block (i, j); the last one is that of the
  // largest parts.
  template <int NPART>
  __device__ void add(int q, int i, int j, u32x4 a, u32x4 b) {
    if (DUAL && q < SplitOrder<NPART>::n - 1)
      low[i][j] = mfma_part<NPART>(a, b, low[i][j]);
    else
      sum[i][j] = mfma_part<NPART>(a, b, sum[i][j]);
  }
  __device__ void finish() {
    if constexpr (DUAL) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) sum[i][j] += low[i][j];
    }
  }
};

// One stage (16 k) of a wave's blocks: rows ra + 32i of the tile against rows
// rb + 32j.
template <int ROWS, int NPART, int MI, int NI, bool DUAL>
__device__ inline void split_stage(const char* tile, int ra, int rb, int l32, int lhi, SplitAcc<MI, NI, DUAL>& acc) {
  using T = SplitTile<ROWS, NPART>;
  using O = SplitOrder<NPART>;
  u32x4 a[MI][NPART];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int p = 0; p < NPART; ++p) a[i][p] = T::get(tile, p, ra + 32 * i + l32, lhi);
#pragma unroll
  for (int j = 0; j < NI; ++j) {
    u32x4 b[NPART];
#pragma unroll
    for (int p = 0; p < NPART; ++p) b[p] = T::get(tile, p, rb + 32 * j + l32, lhi);
#pragma unroll
    for (int q = 0; q < O::n; ++q)
#pragma unroll
      for (int i = 0; i < MI; ++i) acc.template add<NPART>(q, i, j, a[i][O::a[q]], b[O::b[q]]);
  }
}

// The contraction of a workgroup of four waves: two stage buffers at lds, one
// barrier per stage, loads one stage ahead.  load(s): this thread's share of
// stage s to registers (s past the end: anything in range), store(tile):
// those registers to a tile.  ns is even.
template <int ROWS, int NPART, int MI, int NI, bool DUAL, class Load, class Store>
__device__ inline void split_loop4(char* lds, int ns, int ra, int rb, int l32, int lhi, SplitAcc<MI, NI, DUAL>& acc,
                                   Load&& load, Store&& store) {
  using T = SplitTile<ROWS, NPART>;
  load(0);
  store(lds);
  load(1);
  __syncthreads();
  for (int s = 0; s < ns; s += 2) {
    store(lds + T::kBytes);
    load(s + 2);
    __builtin_amdgcn_sched_barrier(0);
    split_stage<ROWS, NPART>(lds, ra, rb, l32, lhi, acc);
    __syncthreads();
    store(lds);
    load(s + 3);
    __builtin_amdgcn_sched_barrier(0);
    split_stage<ROWS, NPART>(lds + T::kBytes, ra, rb, l32, lhi, acc);
    __syncthreads();
  }
  acc.finish();
}

// The contraction of a workgroup of eight waves, waves 0-3 and 4-7 (one of
// each per SIMD) half a stage apart: while four waves read their operands of
// a stage from LDS, the other four run the MFMAs of theirs, and split and
// write (store) the stage two ahead beside them.  Three stage buffers at lds.
template <int ROWS, int NPART, int MI, int NI, bool DUAL, class Load, class Store>
__device__ inline void split_loop8(char* lds, int ns, int ra, int rb, int l32, int lhi, int grp,
                                   SplitAcc<MI, NI, DUAL>& acc, Load&& load, Store&& store) {
  using T = SplitTile<ROWS, NPART>;
  using O = SplitOrder<NPART>;
  load(0);
  store(lds);
  load(1);
  store(lds + T::kBytes);
  load(2);
  __syncthreads();
  if (grp) __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  int cur = 0, nxt = 2 * T::kBytes;
  for (int s = 0; s < ns; ++s) {
    u32x4 fa[MI][NPART], fb[NI][NPART];
    const char* t = lds + cur;
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int p = 0; p < NPART; ++p) fb[j][p] = T::get(t, p, rb + 32 * j + l32, lhi);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int p = 0; p < NPART; ++p) fa[i][p] = T::get(t, p, ra + 32 * i + l32, lhi);
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int q = 0; q < O::n; ++q)
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int i = 0; i < MI; ++i) acc.template add<NPART>(q, i, j, fa[i][O::a[q]], fb[j][O::b[q]]);
    store(lds + nxt);
    load(s + 3);
#pragma unroll
    for (int u = 0; u < O::n * MI * NI; ++u) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one MFMA, then a few vector
      __builtin_amdgcn_sched_group_barrier(0x002, NPART == 3 ? 3 : 6, 0);  // instructions and an LDS write
      __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
    }
    __builtin_amdgcn_s_setprio(0);
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
    cur = cur == 2 * T::kBytes ? 0 : cur + T::kBytes;
    nxt = nxt == 2 * T::kBytes ? 0 : nxt + T::kBytes;
  }
  if (!grp) __builtin_amdgcn_s_barrier();
  acc.finish();
}

}  // namespace hav
