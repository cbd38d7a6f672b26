// Kernels of the delayed first-layer update (include/hieravg.h,
// HIERAVG_UPDATE_DELAYED): within a block of K1 local steps (Algorithm 1,
// Sec. 3.1) every learner of a cluster starts from the same first weight
// block Wb, and after k steps its block is Wb - lr * sum_{k'<k} G_k'^T X_k'.
//
// k_gram:         the Gram blocks X_k X_k'^T (k' < k) of each learner's
//                 minibatches in each block, which turn the forward from Wb
//                 into the forward from the learner's current block.
// (The block's forward and block-end update are in k_split.hip.)
#include <algorithm>

#include "internal.h"

namespace hav {

constexpr int kKC = 64;  // K floats per LDS chunk

// ------------------------------------------------------------ Gram blocks
// One workgroup per (learner p, block b, K split ks): all step pairs k2 < k of
// the block at once.  The K1*Bp minibatch rows of the block (gathered, this
// split's input features) are staged through LDS 64 features at a time, the
// next chunk's loads in flight during the current chunk's MFMAs; each wave
// owns a fixed set of the 16x16 output blocks of the lower block triangle
// (16x16x4 MFMAs, the k permutation of k_fwd_nt).  Every minibatch row is
// read once per split; the consumer adds the KSG partial sums.
constexpr int kGT = 512, kGW = kGT / 64;  // threads and waves per workgroup
constexpr int kGramMaxBlocks = 14;  // 16x16 output blocks per wave (K1 <= 8, Bp <= 32)
template <int NB, int ROWS>
__global__ __launch_bounds__(kGT) void k_gram(const float* __restrict__ X, int64_t ldx, int K,
                                              const int32_t* __restrict__ idx, float* __restrict__ gram, int P,
                                              int K1, int B, int Bp, int KSG) {
  constexpr int kRows = ROWS;         // LDS capacity in rows (K1 * Bp <= ROWS)
  constexpr int kL = kKC + 4;         // LDS row length
  constexpr int kLPT = kRows * (kKC / 4) / kGT;  // 16-byte pieces per thread per chunk (at most)
  __shared__ __attribute__((aligned(16))) float xs[kRows * kL];
  const int ks = blockIdx.x % KSG;
  const int pb = blockIdx.x / KSG;  // p + P * b
  const int p = pb % P, b = pb / P;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: scalar block bookkeeping
  const int lrow = lane & 15, lgrp = lane >> 4;
  const int rows = K1 * Bp;
  const int nch = K / kKC;
  const int c0 = (int)((int64_t)nch * ks / KSG), c1 = (int)((int64_t)nch * (ks + 1) / KSG);
  // Bp is 16 or 32 (B <= 32): row and block indices split with shifts.
  const int lg_bp = Bp == 32 ? 5 : 4, lg_mbs = lg_bp - 4;
  // Row r = k*Bp + s of the block: sample s of step b*K1 + k (rows past B: zero).
  const float* src[kLPT];
  bool ok[kLPT];
  int off[kLPT];
#pragma unroll
  for (int i = 0; i < kLPT; ++i) {
    const int q = tid + kGT * i;
    const int r = q >> 4, c4 = q & 15;
    const int k = r >> lg_bp, sm = r & (Bp - 1);
    ok[i] = r < rows && sm < B;
    const int64_t e = ((int64_t)(b * K1 + (ok[i] ? k : 0)) * P + p) * B + (ok[i] ? sm : 0);
    src[i] = X + (int64_t)idx[e] * ldx + 4 * c4;
    off[i] = (r < kRows ? r : 0) * kL + 4 * c4;
  }
  // Output blocks of this wave: block e = wave + kGW*t over the lower triangle
  // (pair (k, k2), row block mb, column block nb); wave-uniform.
  const int mbs = 1 << lg_mbs;
  const int nblk = K1 * (K1 - 1) / 2 * mbs * mbs;
  int bk[NB], bk2[NB], bmb[NB], bnb[NB];
  int arow[NB], brow[NB];
  bool bon[NB];
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    const int e = wave + kGW * t;
    bon[t] = e < nblk;
    const int ee = bon[t] ? e : 0;
    const int pr = ee >> (2 * lg_mbs), rem = ee & (mbs * mbs - 1);
    int k = 1, k2 = pr;
    while (k2 >= k) {
      k2 -= k;
      ++k;
    }
    bk[t] = k;
    bk2[t] = k2;
    bmb[t] = rem >> lg_mbs;
    bnb[t] = rem & (mbs - 1);
    arow[t] = (k * Bp + 16 * bmb[t] + lrow) * kL + 4 * lgrp;
    brow[t] = (k2 * Bp + 16 * bnb[t] + lrow) * kL + 4 * lgrp;
  }
  const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
  f32x4 acc[NB];
#pragma unroll
  for (int t = 0; t < NB; ++t) acc[t] = zero4;
  f32x4 v[kLPT];
  auto load = [&](int c) {
#pragma unroll
    for (int i = 0; i < kLPT; ++i) v[i] = *(const f32x4*)(src[i] + (int64_t)c * kKC);
  };
  // Piece i holds row (tid >> 4) + 32*i; with B == Bp every staged row is a
  // sample.
  const bool all_rows = B == Bp;
  auto store = [&]() {
    if (all_rows) {
#pragma unroll
      for (int i = 0; i < kLPT; ++i)
        if ((tid >> 4) + 32 * i < rows) *(f32x4*)&xs[off[i]] = v[i];
    } else {
#pragma unroll
      for (int i = 0; i < kLPT; ++i)
        if ((tid >> 4) + 32 * i < rows) *(f32x4*)&xs[off[i]] = ok[i] ? v[i] : zero4;
    }
  };
  if (c0 < c1) {
    load(c0);
    for (int c = c0; c < c1; ++c) {
      store();
      __syncthreads();
      load(c + 1 < c1 ? c + 1 : c);  // next chunk in flight (the last again at the end)
      __builtin_amdgcn_sched_barrier(0);
      // Blocks past nblk repeat block 0 (their sums are not stored): no
      // branch around the MFMAs, so the accumulators stay in place.
#pragma unroll
      for (int t = 0; t < NB; ++t) {
#pragma unroll
        for (int q = 0; q < kKC / 16; ++q) {
          const f32x4 x = *(const f32x4*)&xs[arow[t] + 16 * q];
          const f32x4 y = *(const f32x4*)&xs[brow[t] + 16 * q];
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i], y[i], acc[t], 0, 0, 0);
        }
      }
      __syncthreads();
    }
  }
  // gram[ks][b][p][k][k2][s][s2]
  const int K2n = gridDim.x / (KSG * P);
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    if (!bon[t]) continue;
    float* out = gram + (((((int64_t)ks * K2n + b) * P + p) * K1 + bk[t]) * K1 + bk2[t]) * Bp * Bp +
                 (16 * bmb[t] + 4 * lgrp) * Bp + 16 * bnb[t] + lrow;
#pragma unroll
    for (int r = 0; r < 4; ++r) out[r * Bp] = acc[t][r];
  }
}

// gram[0] += gram[1] + ... + gram[KSG-1] over the blocks k2 < k (added in
// split order), so the consumer reads one sum.  Element i enumerates
// (block and learner bp, step pair, 16-byte piece q of the Bp x Bp block).
__global__ __launch_bounds__(256) void k_gram_reduce(float* __restrict__ gram, int64_t split, int64_t n4, int K1,
                                                     int pairs, int blk4, int KSG) {
  f32x4* g = (f32x4*)gram;
  const int64_t s4 = split / 4;
  for (int64_t i = blockIdx.x * 256ll + threadIdx.x; i < n4; i += (int64_t)gridDim.x * 256) {
    const int q = (int)(i % blk4);
    const int64_t t = i / blk4;
    const int pr = (int)(t % pairs);
    const int64_t bp = t / pairs;
    int k = 1, k2 = pr;
    while (k2 >= k) {
      k2 -= k;
      ++k;
    }
    const int64_t o = ((bp * K1 + k) * K1 + k2) * blk4 + q;
    f32x4 v = g[o];
    for (int t2 = 1; t2 < KSG; ++t2) v += g[t2 * s4 + o];
    g[o] = v;
  }
}

#ifndef HAV_GRAM_TARGET
#define HAV_GRAM_TARGET 512
#endif
int gram_splits(int P, int K2, int K) {
  // about two workgroups per CU, at least two 64-wide chunks per split
  const int target = HAV_GRAM_TARGET;
  int ksg = (target + P * K2 - 1) / (P * K2);
  return std::max(1, std::min(ksg, K / kKC / 2));
}

void launch_gram(hipStream_t s, const float* X, int64_t ldx, int K, const int32_t* idx, float* gram, int P, int K1,
                 int K2, int B, int Bp, int KSG) {
  const int nblk = K1 * (K1 - 1) / 2 * (Bp / 16) * (Bp / 16);
  if (nblk == 0 || (Bp != 16 && Bp != 32)) return;  // the delayed schedule has B <= 32
  const unsigned grid = (unsigned)((int64_t)P * K2 * KSG);
  const int nb = (nblk + kGW - 1) / kGW;
#define HAV_GRAM(N_, R_) launch(k_gram<N_, R_>, grid, kGT, 0, s, X, ldx, K, idx, gram, P, K1, B, Bp, KSG)
  if (K1 * Bp <= 128) {
    if (nb <= 1)
      HAV_GRAM(1, 128);
    else if (nb <= 3)
      HAV_GRAM(3, 128);
    else
      HAV_GRAM(6, 128);
  } else {
    if (nb <= 6)
      HAV_GRAM(6, 256);
    else
      HAV_GRAM(kGramMaxBlocks, 256);
  }
#undef HAV_GRAM
}

void launch_gram_reduce(hipStream_t s, float* gram, int P, int K1, int K2, int Bp, int KSG) {
  const int64_t split = (int64_t)K2 * P * K1 * K1 * Bp * Bp;
  const int pairs = K1 * (K1 - 1) / 2, blk4 = Bp * Bp / 4;
  const int64_t n4 = (int64_t)K2 * P * pairs * blk4;
  const int64_t g = std::min<int64_t>((n4 + 255) / 256, 2048);
  launch(k_gram_reduce, (unsigned)g, 256, 0, s, gram, split, n4, K1, pairs, blk4, KSG);
}

}  // namespace hav
