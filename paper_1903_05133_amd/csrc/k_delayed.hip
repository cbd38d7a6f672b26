// The wide contractions of a round as split float32 products (split.h), and
// the kernels of the delayed first-layer update (include/hieravg.h,
// HIERAVG_UPDATE_DELAYED): within a block of K1 local steps (Algorithm 1,
// Sec. 3.1) every learner of a cluster starts from the same first weight
// block Wb, and after k steps its block is Wb - lr * sum_{k'<k} G_k'^T X_k'.
//
// k_gram:         the Gram blocks X_k X_k'^T (k' < k) of each learner's
//                 minibatches in each block, which turn the forward from Wb
//                 into the forward from the learner's current block.
// k_fwd_split:    part[ks][p][m][n] = sum_{k in split ks} A_p[m][k] * W_p[n][k]
//                 (the forward of either layer; the layouts of FwdArgs).
// k_block_update: the block-end update of the delayed schedule, one GEMM per
//                 cluster (BlkArgs).
// k_gram_split:   the Gram blocks of minibatches of more than 32 samples.
#include <algorithm>

#include "split.h"

namespace hav {

constexpr int kKC = 64;  // K floats per LDS chunk (k_gram) and per chunk of a split

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

// ------------------------------------------------------------ forward
// Workgroup tile BM rows (samples) x BN columns (units), one K split; wave
// tile WM x WN.  The tile's rows of both operands are read 16 k at a time
// with 16-byte loads (four lanes per row), one stage ahead in registers, and
// go to LDS as three bf16 or two f16 parts (the loops of split.h).  FULL: every
// row and column in range.  DUAL: a second set of sums for the small products
// (SplitAcc): in every form but the two parts of a delayed block, which replaced
// 32x32x2 float32 MFMAs and round less than half as often with one set; there
// the registers of a second one leave the 128 x 256 tile one workgroup per CU
// (288 workgroups, 16 x 320 rows, 448 units, 1104 features: 33 -> 42 us).
template <int BM, int BN, int WM, int WN, int NPART, int ASRC, bool FULL, bool DUAL, int WPE>
__global__ __launch_bounds__(64 * (BM / WM) * (BN / WN)) __attribute__((amdgpu_waves_per_eu(WPE))) void k_fwd_split(
    FwdArgs a, int ntiles, int mtiles) {
  constexpr int NTH = 64 * (BM / WM) * (BN / WN);
  constexpr int ROWS = BM + BN, RPP = NTH / 4, NP = (ROWS + RPP - 1) / RPP;  // pieces per thread, rows per pass
  constexpr int MI = WM / 32, NI = WN / 32;
  using T = SplitTile<ROWS, NPART>;
  __shared__ __attribute__((aligned(16))) char lds[NTH == 512 ? 3 : 2][T::kBytes];
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  const int q1 = qdiv_small(bid, ntiles, qdiv_inv(ntiles)), nt = bid - q1 * ntiles;
  const int q2 = qdiv_small(q1, mtiles, qdiv_inv(mtiles)), mt = q1 - q2 * mtiles;
  const int g = qdiv_small(q2, a.KS, qdiv_inv(a.KS)), ks = q2 - g * a.KS;
  const int GM = a.SG * a.Mp;
  const int nch = a.K / kKC;
  const int c0 = ks * a.cps, c1 = min(nch, c0 + a.cps);
  const int ns = 4 * (c1 - c0);  // stages
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, lhi = lane >> 5;
  const int wm = wave / (BN / WN) * WM, wn = wave % (BN / WN) * WN;
  const int mbase = mt * BM, nbase = nt * BN;
  const int sr = tid >> 2, sq = tid & 3;

  // Whether this thread's row of pass i is one of A's (the same for a wave).
  auto is_a = [&](int i) { return RPP * (i + 1) <= BM || (RPP * i < BM && sr + RPP * i < BM); };
  auto none = [&](int i) { return RPP * (i + 1) > ROWS && sr + RPP * i >= ROWS; };  // no row for this thread
  const float* src[NP];
  bool ok[NP];
  int ex[NP];  // two parts: the row's power-of-two scale
  const float* wp = a.W + (int64_t)(g / a.wdiv) * a.w_pitch;
  const uint32_t* wmax = NPART == 2 ? a.wmax + (int64_t)(g / a.wdiv) * a.wmax_pitch : nullptr;
  const float inv_mp = qdiv_inv(a.Mp), inv_vs = qdiv_inv(a.vS > 0 ? a.vS : 1);
  // Row m of the group's A; past its samples (not valid: zeros) row 0's.
  auto a_row = [&](int m, bool& valid, float inv_mp, float inv_vs) {
    const int jj = qdiv_small(m, a.Mp, inv_mp), sm = m - jj * a.Mp;
    valid = FULL || (m < GM && sm < a.M);
    const int v = valid ? jj : 0;
    int64_t p = (int64_t)g * a.SG + v;
    if (a.vS > 0) {
      const int k = qdiv_small(v, a.vS, inv_vs);
      p = (int64_t)k * a.P + (int64_t)g * a.vS + (v - k * a.vS);
    }
    const int sc = valid ? sm : 0;
    return a.A + (ASRC == A_GATHER ? (int64_t)a.idx[p * a.M + sc] : p * a.Mp + sc) * a.lda;
  };
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    if (none(i)) continue;
    const int r = sr + RPP * i;
    if (is_a(i)) {
      src[i] = a_row(mbase + r, ok[i], inv_mp, inv_vs) + 4 * sq;
      ex[i] = a.xexp;
    } else {
      const int n = nbase + r - BM;
      ok[i] = true;  // columns past N repeat row 0 and are not stored
      const int nc = FULL || n < a.N ? n : 0;
      src[i] = wp + (int64_t)nc * a.ldw + 4 * sq;
      if (NPART == 2) ex[i] = split_exp(wmax[nc]);
    }
    src[i] += (int64_t)c0 * kKC;
  }
  f32x4 v[NP];
  auto load = [&](int s) {  // past the end: the last stage again, unused
    const int o = 16 * min(s, ns - 1);
#pragma unroll
    for (int i = 0; i < NP; ++i)
      if (!none(i)) v[i] = *(const f32x4*)(src[i] + o);
  };
  auto store = [&](char* tile) {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      if (none(i)) continue;
      f32x4 x = v[i];
      if (is_a(i)) {
        if (!FULL && !ok[i]) x = f32x4{0.f, 0.f, 0.f, 0.f};
        if (ASRC == A_RELU) {  // NaN stays NaN
          x.x = x.x < 0.0f ? 0.0f : x.x;
          x.y = x.y < 0.0f ? 0.0f : x.y;
          x.z = x.z < 0.0f ? 0.0f : x.z;
          x.w = x.w < 0.0f ? 0.0f : x.w;
        }
      }
      if (NPART == 2) {
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = __builtin_amdgcn_ldexpf(x[e], ex[i]);
      }
      T::put4(tile, sr + RPP * i, sq, x);
    }
  };
  SplitAcc<MI, NI, DUAL> acc;
  acc.clear();

  if constexpr (NTH == 512)
    split_loop8<ROWS, NPART>(lds[0], ns, wm, BM + wn, l32, lhi, wave >> 2, acc, load, store);
  else
    split_loop4<ROWS, NPART>(lds[0], ns, wm, BM + wn, l32, lhi, acc, load, store);

  // Infinite operands: one of their parts is NaN, and so is every sum that they
  // enter.  Which sums those are is noted here, and they are taken again, as
  // float32 gives them, after the others are stored (their code and registers
  // stay out of the way).
  auto nan = [](float x) { return x != x; };
  uint32_t cols[NI];  // gathered rows: columns with a NaN; hidden ones: blocks i with a NaN
#pragma unroll
  for (int j = 0; j < NI; ++j) {
    cols[j] = 0;
    if constexpr (ASRC == A_GATHER) {
      // dataset rows are finite: a column's weights make NaN of every row
      cols[j] = __builtin_amdgcn_readfirstlane((uint32_t)__ballot(nan(acc.sum[0][j][0])));
    } else {
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        float t = 0.0f;
#pragma unroll
        for (int r = 0; r < 16; ++r) t += acc.sum[i][j][r];
        cols[j] |= __any(nan(t)) ? 1u << i : 0u;
      }
    }
  }

  int en[NI];  // two parts: minus the scales of the lane's columns
#pragma unroll
  for (int j = 0; j < NI; ++j)
    en[j] = NPART == 2 ? -a.xexp - split_exp(wmax[min(nbase + wn + 32 * j + l32, a.N - 1)]) : 0;
  const int64_t PT = a.PT > 0 ? a.PT : a.P;
  const int64_t gbase = a.vS > 0 ? (int64_t)g * a.vS : (int64_t)g * a.SG;
  const int64_t kstride = a.vS > 0 ? a.P : 0;
  // (computed again: the loop's registers are at the limit of their occupancy)
  int mp2 = a.Mp, vs2 = a.vS > 0 ? a.vS : 1;
  asm volatile("" : "+s"(mp2), "+s"(vs2));
  const float inv_mp2 = qdiv_inv(mp2), inv_vs2 = qdiv_inv(vs2);
  auto out = [&](int row) {  // row of the group -> its partial sums
    const int mv = qdiv_small(row, a.Mp, inv_mp2), sm = row - mv * a.Mp;
    const int vk = a.vS > 0 ? qdiv_small(mv, a.vS, inv_vs2) : 0, vj = a.vS > 0 ? mv - vk * a.vS : mv;
    return a.part + (((int64_t)ks * PT + vk * kstride + gbase + vj) * a.Mp + sm) * a.N;
  };
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    // The lane's rows 8t + e (e < 4) share one member (Mp is a multiple of 16).
    const int mrow = mbase + wm + 32 * i + 4 * lhi;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int row = mrow + 8 * t;
      if (!FULL && row >= GM) continue;
      float* dst = out(row) + nbase + wn + l32;
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        if (!FULL && nbase + wn + 32 * j + l32 >= a.N) continue;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          dst[(int64_t)e * a.N + 32 * j] =
              NPART == 2 ? __builtin_amdgcn_ldexpf(acc.sum[i][j][4 * t + e], en[j]) : acc.sum[i][j][4 * t + e];
      }
    }
  }

#pragma unroll
  for (int j = 0; j < NI; ++j) {
    if (__builtin_expect(cols[j] == 0, 1)) continue;
    if constexpr (ASRC == A_GATHER) {
      // Only the column's infinite weights count (with a NaN weight the sums are
      // right as they are): the wave looks for them together, then takes one row
      // of either half at a time.
      for (uint32_t left = cols[j]; left; left &= left - 1) {
        const int col = nbase + wn + 32 * j + __builtin_ctz(left);
        if (col >= a.N) break;
        const float* w = wp + (int64_t)col * a.ldw;
        bool inf = false, nans = false;
        for (int k = c0 * kKC; k < c1 * kKC && !nans; k += 64) {
          const float v = w[k + l32 + 32 * lhi];
          nans = __any(nan(v));
          inf = inf || __any(__builtin_isinf(v));
        }
        if (nans || !inf) continue;
        for (int q = 0; q < 16 * MI; ++q) {
          const int row = mbase + wm + 8 * (q >> 2) + 4 * lhi + (q & 3);
          bool valid;
          const float* x = a_row(row, valid, inv_mp2, inv_vs2);
          float s = 0.0f;
          bool all = false;  // NaN in both halves
          for (int k = c0 * kKC; k < c1 * kKC && !all; k += 64)
            for (uint64_t b = __ballot(__builtin_isinf(w[k + l32 + 32 * lhi])); b && !all; b &= b - 1) {
              const int kk = k + __builtin_ctzll(b);
              s = __builtin_fmaf(valid ? x[kk] : 0.0f, w[kk], s);
              all = __all(nan(s));
            }
          if (l32 == __builtin_ctz(left) && (FULL || row < GM)) out(row)[col] = s;
        }
      }
    } else {
      // Hidden values may be infinite too: every term again, lane by lane (row m
      // of a group is row m of its block; vS = 0).  A finite sum had no infinite
      // operand and stays.
      const int col = nbase + wn + 32 * j + l32;
      const float* w = wp + (int64_t)min(col, a.N - 1) * a.ldw;
      for (int q = 0; q < 16 * MI; ++q) {
        if (!(cols[j] >> (q >> 4) & 1)) continue;
        const int row = mbase + wm + 8 * (q >> 2) + 4 * lhi + (q & 3);
        const float* x = a.A + ((int64_t)g * GM + min(row, GM - 1)) * a.lda;
        float s = 0.0f;
        for (int k = c0 * kKC; k < c1 * kKC && !nan(s); ++k)
          s = __builtin_fmaf(x[k] < 0.0f ? 0.0f : x[k], w[k], s);
        if (!__builtin_isfinite(s) && row < GM && col < a.N) out(row)[col] = s;
      }
    }
  }
}

// The tile of a forward over `groups` row groups of GM rows each.
//  - 256 x 256 for the forward of a delayed block where the operands are long:
//    with the split count that brings the grid to one workgroup per CU, 1024 k
//    and more per split (a 512-row group against 1024 units over 150528
//    features: 2.24 ms = 282 TFLOP/s, with 128 x 256 tiles 2.47; over 3072
//    features the 128 x 256 tile is as fast with half the splits); the other
//    forwards take two sets of sums, which this tile's registers do not hold;
//  - 128 x 256 where at least 32 such tiles exist, so that 8 splits fill the
//    GPU (2048 rows, 512 units, 3072 features in two parts: 28.6 us, 31.8 us
//    with 128 x 128 tiles; the float32 MFMA form took 66);
//  - fewer rows per group: 128 x 128 (8 x 128 rows: 25.5 us against 28.4; 58
//    in float32), 64 x 128 (8 x 64 rows: 20 us against 21.6 with 128 rows;
//    29 in float32), 32 x 128 (four workgroups per CU: 64 x 32 rows against 192
//    units over 3072 features 33.3 us, two per CU 38.6, 38.1 in float32; at 64
//    rows two are faster, 28.4 us against 33.0 for 64 x 64 rows, 128 units).
enum FwdTile { FT_256, FT_128x256, FT_128, FT_64, FT_32 };
struct FwdTileShape {
  int bm, bn, wgs;  // rows, columns, workgroups a launch aims for
};
static constexpr FwdTileShape kFwdTiles[] = {
    {256, 256, 256}, {128, 256, 256}, {128, 128, 256}, {64, 128, 512}, {32, 128, 1024}};
static int64_t fwd_tiles(FwdTile t, int64_t groups, int GM, int N) {
  return groups * ((GM + kFwdTiles[t].bm - 1) / kFwdTiles[t].bm) * ((N + kFwdTiles[t].bn - 1) / kFwdTiles[t].bn);
}
static FwdTile fwd_tile(int64_t groups, int GM, int N, int K, bool block) {
  if (block && GM % 256 == 0 && N % 256 == 0) {
    const int64_t ks = (256 + fwd_tiles(FT_256, groups, GM, N) - 1) / fwd_tiles(FT_256, groups, GM, N);
    if (K / ks >= 1024) return FT_256;
  }
  if (GM > 64) return N > 128 && fwd_tiles(FT_128x256, groups, GM, N) >= 32 ? FT_128x256 : FT_128;
  return GM > 32 ? FT_64 : FT_32;
}

void plan_split(int groups, int GM, int N, int K, bool block, int* KS, int* cps) {
  const int nch = K / kKC;
  if (!fwd_split_takes(groups, GM, N, K)) {
    plan_split_nt(groups, GM, N, K, KS, cps);
    return;
  }
  const FwdTile t = fwd_tile(groups, GM, N, K, block);
  const int64_t tiles = fwd_tiles(t, groups, GM, N);
  // With two sets of sums one workgroup of the 128 x 256 tile fits a CU, and two
  // of the 128 x 128 one slow each other: no more than one per CU, then (3327
  // rows, 448 units, 2816 features, twice: 194 us with 208 workgroups, 254 with
  // 260; 3002 rows, 128 units, 7104 features: 177 with 240, 194 with 264).
  const bool at_most = !block && (t == FT_128x256 || t == FT_128);
  auto splits = [&](int64_t wgs) { return std::max<int64_t>(1, (at_most ? wgs : wgs + tiles - 1) / tiles); };
  // Past 8 splits the partial sums cost more than two more workgroups per CU
  // give (softmax, 8 learners, 7776 features, 97 classes: 2.41 ms a job with one
  // split per 64 features, 1.85 with one per 128).
  const int64_t want = t == FT_32 ? std::min(splits(kFwdTiles[t].wgs), std::max<int64_t>(8, splits(512)))
                                  : splits(kFwdTiles[t].wgs);
  int ks = (int)std::min<int64_t>(nch, want);
  const int c = (nch + ks - 1) / ks;
  *KS = (nch + c - 1) / c;
  *cps = c;
}

void launch_fwd(hipStream_t s, const FwdArgs& a, ASource src) {
  const int GM = a.SG * a.Mp;
  const int groups = a.vS > 0 ? a.P / a.vS : a.P / a.SG;
  if (!fwd_split_takes(groups, GM, a.N, a.K)) {
    launch_fwd_nt(s, a, src);
    return;
  }
#define HAV_FS1(BM_, BN_, WM_, WN_, WPE_, NPART_, SRC_, FULL_, DUAL_)                                           \
  launch(k_fwd_split<BM_, BN_, WM_, WN_, NPART_, SRC_, FULL_, DUAL_, WPE_>,                                     \
         (unsigned)((int64_t)groups * a.KS * ((GM + BM_ - 1) / BM_) * ((a.N + BN_ - 1) / BN_)),                 \
         64 * (BM_ / WM_) * (BN_ / WN_), 0, s, a, (a.N + BN_ - 1) / BN_, (GM + BM_ - 1) / BM_)
#define HAV_FS2(BM_, BN_, WM_, WN_, WPE_, NPART_, DUAL_)                                                        \
  do {                                                                                                          \
    if (GM % BM_ == 0 && a.N % BN_ == 0 && a.M == a.Mp)                                                         \
      HAV_FS1(BM_, BN_, WM_, WN_, WPE_, NPART_, A_GATHER, true, DUAL_);                                         \
    else                                                                                                        \
      HAV_FS1(BM_, BN_, WM_, WN_, WPE_, NPART_, A_GATHER, false, DUAL_);                                        \
  } while (0)
#define HAV_FS(BM_, BN_, WM_, WN_, WPE_)                                                                        \
  do {                                                                                                          \
    if (src == A_RELU)                                                                                          \
      HAV_FS1(BM_, BN_, WM_, WN_, WPE_, 3, A_RELU, false, true);                                                \
    else if (!a.wmax)                                                                                           \
      HAV_FS2(BM_, BN_, WM_, WN_, WPE_, 3, true);                                                               \
    else if (a.vS > 0)                                                                                          \
      HAV_FS2(BM_, BN_, WM_, WN_, WPE_, 2, false);                                                              \
    else                                                                                                        \
      HAV_FS2(BM_, BN_, WM_, WN_, WPE_, 2, true);                                                               \
  } while (0)
  switch (fwd_tile(groups, GM, a.N, a.K, a.vS > 0)) {
    case FT_256: HAV_FS2(256, 256, 128, 64, 2, 2, false); break;
    case FT_128x256: HAV_FS(128, 256, 64, 64, 2); break;
    case FT_128: HAV_FS(128, 128, 64, 32, 2); break;
    case FT_64: HAV_FS(64, 128, 64, 32, 3); break;
    default: HAV_FS(32, 128, 32, 32, 4); break;
  }
#undef HAV_FS2
#undef HAV_FS
#undef HAV_FS1
}

// ------------------------------------------------------------ block update
// Wo_g = base_g - lr_eff * sum_r G[r][:]^T X[r][:] (BlkArgs), workgroup tile
// BM units x BN inputs of one group's block, contracted over the group's
// R = K1*SG*B rows 16 at a time.  A lane loads one or two columns of eight rows
// (a wave instruction reads consecutive columns of a row, whose address is
// scalar, from the row tables) and writes each column's eight values as one
// 16-byte piece per part: the transposition that the MFMA operands need costs
// nothing.  Two columns halve the load instructions, whose address processing
// (16 cycles each for any width) kept the texture units 0.7 busy (512 x 3072, four
// groups of 512 rows: 40.4 -> 37.8 us; with heavy-ball 53 -> 50).
template <int BM, int BN, int WM, int WN, bool FULL, int WPE>
__global__ __launch_bounds__(64 * (BM / WM) * (BN / WN)) __attribute__((amdgpu_waves_per_eu(WPE))) void k_block_update(
    BlkArgs a, const uint32_t* __restrict__ gtab, const uint32_t* __restrict__ xtab, int mtiles, int ntiles) {
  constexpr int NW = (BM / WM) * (BN / WN), NTH = 64 * NW;
  constexpr int VW = BM % 128 == 0 && BN % 128 == 0 ? 2 : 1;  // columns per lane
  constexpr int ROWS = BM + BN, UC = 64 * VW, UG = BM / UC, UX = BN / UC;  // UC-column groups of G and X
  constexpr int UT = 2 * (UG + UX), NU = (UT + NW - 1) / NW;  // (row half, column group) units, per wave
  constexpr int MI = WM / 32, NI = WN / 32;
  static_assert(NW % 2 == 0, "a wave's units share their row half");
  using T = SplitTile<ROWS, 2>;
  __shared__ int gexp[BM];  // the scales of the tile's units
  __shared__ __attribute__((aligned(16))) char lds[NTH == 512 ? 3 : 2][T::kBytes];
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  const int mt = bid % mtiles;
  const int nt = (bid / mtiles) % ntiles;
  const int g = bid / (ntiles * mtiles);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, lhi = lane >> 5;
  const int mrow0 = mt * BM, ncol0 = nt * BN;
  const int wm = wave / (BN / WN) * WM, wn = wave % (BN / WN) * WN;
  const int R = a.K1 * a.SG * a.B;
  const int Rp = (R + 31) / 32 * 32, ns = Rp / 16;  // even
  const uint32_t* gt = gtab + (int64_t)g * Rp;
  const uint32_t* xt = xtab + (int64_t)g * Rp;
  if (a.tail && mt == 0) {
    f32x4* Tl = (f32x4*)a.tail + (int64_t)g * a.SG * (a.tail_pitch / 4);
    const int64_t p4 = a.tail_pitch / 4, n4 = a.tail_len / 4, per = (n4 + ntiles - 1) / ntiles;
    const int64_t i1 = min(n4, (nt + 1) * per);
    for (int64_t i = nt * per + tid; i < i1; i += NTH) {
      f32x4 sum = Tl[i];
      for (int j = 1; j < a.SG; ++j) sum += Tl[j * p4 + i];
      const f32x4 mean = sum / (float)a.SG;
      for (int j = 0; j < a.SG; ++j) Tl[j * p4 + i] = mean;
    }
  }
  // Unit u = wave + NW*i of a stage: row half u & 1, column group u >> 1
  // (the groups of G first).
  const int rh = wave & 1;
  float v[NU][8][VW];
  // Row offsets of the next stage to load, read (scalar) a stage ahead.
  uint32_t tg[8], tx[8];
  auto load_tab = [&](int s) {
    const int r0 = 16 * min(s, ns - 1) + 8 * rh;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      tg[e] = gt[r0 + e];
      tx[e] = xt[r0 + e];
    }
  };
  auto load = [&](int s) {
    const int r0 = 16 * min(s, ns - 1) + 8 * rh;  // past the end: the last stage again, unused
#pragma unroll
    for (int i = 0; i < NU; ++i) {
      if (NU * NW > UT && wave + NW * i >= UT) continue;
      const int cg = (wave + NW * i) >> 1;
      const bool isg = NW * i / 2 < UG && ((NW * (i + 1) - 1) / 2 < UG || cg < UG);
      const float* base = isg ? a.G : a.X;
      const int col = (isg ? mrow0 + UC * cg : ncol0 + UC * (cg - UG)) + VW * lane;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        // A row's range ends at its last column, and is empty for an error
        // row past the contraction: what lies outside reads 0.
        const int bytes = isg ? (r0 + e < R ? 4 * a.Mrows : 0) : 4 * a.Ncols;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float*>(base) + ((uint64_t)(isg ? tg[e] : tx[e]) << 6), 0, bytes, 0x00020000);
        if constexpr (VW == 2) {
          const f32x2 x = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(rs, 4 * col, 0, 0));
          v[i][e][0] = x.x;
          v[i][e][1] = x.y;
        } else {
          v[i][e][0] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, 4 * col, 0, 0));
        }
      }
    }
    load_tab(s + 1);
  };
  SplitAcc<MI, NI, false> acc;
  acc.clear();

  load_tab(0);
  const int voff = 4 * (4 * lhi * (int)a.ldw + l32), ld4 = 4 * (int)a.ldw;
  const float* Wb = a.Wb + (int64_t)(g / a.base_div) * a.nbase * a.wb_pitch;
  // Blocks of 32 rows and of 32 columns are whole (both sizes are multiples of 64).
  auto in = [&](int b) {
    return FULL || (mrow0 + wm + 32 * (b / NI) < a.Mrows && ncol0 + wn + 32 * (b % NI) < a.Ncols);
  };
  auto rsrc = [&](const float* base, int b) {
    return buf_rsrc(base + (int64_t)(mrow0 + wm + 32 * (b / NI)) * a.ldw + ncol0 + wn, 32ull * (uint64_t)a.ldw * 4);
  };
  auto soff = [&](int b, int r) { return (8 * (r >> 2) + (r & 3)) * ld4 + 128 * (b % NI); };
  auto ld = [&](const float* base, int b, float (&u)[16]) {
    if (!in(b)) return;
    const __amdgpu_buffer_rsrc_t rs = rsrc(base, b);
#pragma unroll
    for (int r = 0; r < 16; ++r)
      u[r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, voff, soff(b, r), 0));
  };
  constexpr int NB = MI * NI, NQ = NB < 3 ? NB : 3;  // blocks, and those in flight
  float w[NQ][16];
  for (int i = tid; i < BM; i += NTH) {
    const int m = min(mrow0 + i, a.Mrows - 1);
    uint32_t e = 0;
#pragma unroll 4
    for (int c = 0; c < a.gm_n; ++c) e = max(e, a.gmax[((int64_t)g * a.gm_n + c) * a.Mrows + m]);
    if (a.hb) {  // the errors carry their step's coefficient
      float f = 0.0f;
      for (int k = 0; k < a.K1; ++k) f = fmaxf(f, fabsf(a.hb[a.hb_g + k]));
      e = __builtin_bit_cast(uint32_t, __builtin_bit_cast(float, e) * f);
    }
    gexp[i] = split_exp(e);
  }
  __syncthreads();
  int ex[NU][VW];
#pragma unroll
  for (int i = 0; i < NU; ++i)
#pragma unroll
    for (int x = 0; x < VW; ++x) {
      const int cg = (wave + NW * i) >> 1;
      ex[i][x] = cg < UG ? gexp[UC * cg + VW * lane + x] : a.xexp;
    }
  auto store = [&](char* tile) {
#pragma unroll
    for (int i = 0; i < NU; ++i) {
      if (NU * NW > UT && wave + NW * i >= UT) continue;
#pragma unroll
      for (int x = 0; x < VW; ++x) {
        float u[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) u[e] = __builtin_amdgcn_ldexpf(v[i][e][x], ex[i][x]);
        T::put8(tile, UC * ((wave + NW * i) >> 1) + VW * lane + x, rh, u);
      }
    }
  };

  if constexpr (NTH == 512)
    split_loop8<ROWS, 2>(lds[0], ns, wm, BM + wn, l32, lhi, wave >> 2, acc, load, store);
  else
    split_loop4<ROWS, 2>(lds[0], ns, wm, BM + wn, l32, lhi, acc, load, store);

  // Units with infinite errors: as in the forward, from those errors alone (the
  // dataset rows are finite).
  auto nan = [](float x) { return x != x; };
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    if (!__any(gexp[wm + 32 * i + l32] == kNonFiniteExp)) continue;
    for (int u = 0; u < 32; ++u) {
      const int m = mrow0 + wm + 32 * i + u;
      if (gexp[wm + 32 * i + u] != kNonFiniteExp || m >= a.Mrows) continue;
      auto err = [&](int r) { return r < R ? a.G[((uint64_t)gt[r] << 6) + m] : 0.0f; };
      bool inf = false, nans = false;
      for (int r = 0; r < R && !nans; r += 64) {
        const float e = err(r + lane);
        nans = __any(nan(e));
        inf = inf || __any(__builtin_isinf(e));
      }
      if (nans || !inf) continue;
      float s[NI];
#pragma unroll
      for (int j = 0; j < NI; ++j) s[j] = 0.0f;
      bool all = false;
      for (int r0 = 0; r0 < R && !all; r0 += 64)
        for (uint64_t b = __ballot(__builtin_isinf(err(r0 + lane))); b && !all; b &= b - 1) {
          const int r = r0 + __builtin_ctzll(b);
          all = true;
#pragma unroll
          for (int j = 0; j < NI; ++j) {
            const int n = min(ncol0 + wn + 32 * j + l32, a.Ncols - 1);
            s[j] = __builtin_fmaf(err(r), a.X[((uint64_t)xt[r] << 6) + n], s[j]);
            all = all && __all(nan(s[j]));
          }
        }
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (8 * (r >> 2) + 4 * lhi + (r & 3) == u) acc.sum[i][j][r] = s[j];
    }
  }
  // Straight from the accumulators: lane (l, h) holds column l of rows
  // 8t + 4h + e of each 32 x 32 block, so an instruction reads or writes two
  // 128-byte row segments.  Buffer accesses: one lane offset for the whole
  // tile, scalar offsets for the rows; the base of the blocks ahead is in
  // flight.
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int b = 0; b < NQ; ++b) ld(Wb, b, w[b]);
  const float c1 = a.hb ? a.hb[a.hb_c1] : 1.0f, c2 = a.hb ? a.hb[a.hb_c2] : 0.0f;
  const float c3 = a.hb ? 1.0f / a.lr_div : -(*a.lr / a.lr_div);
  uint32_t mx[16];  // magnitudes as bits: NaN and infinity are the largest
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int i = b / NI, j = b % NI;
    float (&x)[16] = w[b % NQ];
    if (in(b)) {
      float u[16];
      if (a.nbase > 1) {  // the mean of the bases, added in order
        for (int c = 1; c < a.nbase; ++c) {
          ld(Wb + (int64_t)c * a.wb_pitch, b, u);
#pragma unroll
          for (int r = 0; r < 16; ++r) x[r] += u[r];
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) x[r] = x[r] / (float)a.nbase;
      }
      // The change from the base (what the errors give, and c2 times the mean
      // of B2) is summed first, so that the result is rounded to the base's
      // precision once, in the fma that scales the base.
      float d[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int er = -a.xexp - gexp[wm + 32 * i + 8 * (r >> 2) + 4 * lhi + (r & 3)];  // minus the scales
        d[r] = c3 * __builtin_amdgcn_ldexpf(acc.sum[i][j][r], er);
      }
      if (a.hb && a.B2) {
        const float* b2 = a.B2 + (int64_t)g * a.b2_rows * a.b2_pitch;
        float bm[16];
        ld(b2, b, bm);
        for (int c = 1; c < a.b2_rows; ++c) {
          ld(b2 + (int64_t)c * a.b2_pitch, b, u);
#pragma unroll
          for (int r = 0; r < 16; ++r) bm[r] += u[r];
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) d[r] += c2 * (bm[r] / (float)a.b2_rows);
      }
      const __amdgpu_buffer_rsrc_t rs = rsrc(a.Wo + (int64_t)g * a.wo_pitch, b);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        x[r] = __builtin_fmaf(c1, x[r], d[r]);
        const uint32_t m = __builtin_bit_cast(uint32_t, x[r]) & 0x7fffffffu;
        mx[r] = j == 0 ? m : max(mx[r], m);
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x[r]), rs, voff, soff(b, r), 0);
      }
    }
    if (b + NQ < NB) ld(Wb, b + NQ, x);
    if (j == NI - 1 && a.wmax_out && in(b - j)) {
      // Row maxima over the wave's columns: over 16 lanes by DPP moves, then
      // lane l takes row l % 16 of its half.  Only a value above what the
      // table holds goes out (a few per row in a launch).
      uint32_t mine = 0;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const uint32_t m = max16(mx[r]);
        if ((lane & 15) == r) mine = m;
      }
      const int r = lane & 15;
      uint32_t* d = a.wmax_out + (int64_t)g * a.Mrows + mrow0 + wm + 32 * i + 8 * (r >> 2) + 4 * lhi + (r & 3);
      if (mine > __hip_atomic_load(d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(d, mine);
    }
  }
}

// Tiles of the block update: 256 x 256 in eight waves where they waste no units,
// the contraction is 256 rows and more (a short one is the stream of W and the
// buffers, which needs more workgroups per CU: 40 buffers of 128 x 8832, 32
// rows, a whole job 6.6 ms in float32, 7.0 with this tile, 5.0 with 128 x 128,
// 5.6 with 64 x 64) and the grid holds two of them per CU and more (1024 x
// 150528, four groups of 512 rows: 2.36 ms = 268 TFLOP/s, as 128 x 256 in four
// waves; 128 x 128 2.6, the float32 MFMA form 4.8; the matrix cores are busy 35 %
// of the cycles at 2.0 GHz, the waves wait 47 %); else 128 x 128 (512 x 3072, four groups: 38 us against 57
// with 64 x 64 tiles, 66 in float32) down to 256 workgroups, and 64 x 64 for
// smaller blocks (320 x 1024, two groups of 243 rows: 11 us against 19, 14.6 in
// float32; 512 x 3072, two groups of 2048 rows: 99 us against 115).
void launch_block_update(hipStream_t s, const BlkArgs& a) {
  const int groups = a.P / a.SG;
  auto tiles = [&](int bm, int bn) { return (int64_t)groups * ((a.Mrows + bm - 1) / bm) * ((a.Ncols + bn - 1) / bn); };
#define HAV_BU(BM_, BN_, WM_, WN_, WPE_)                                                                       \
  do {                                                                                                         \
    const int mt = (a.Mrows + BM_ - 1) / BM_, nt = (a.Ncols + BN_ - 1) / BN_;                                  \
    const unsigned grid = (unsigned)((int64_t)groups * mt * nt);                                               \
    constexpr int th = 64 * (BM_ / WM_) * (BN_ / WN_);                                                         \
    if (a.Mrows % BM_ == 0 && a.Ncols % BN_ == 0)                                                              \
      launch(k_block_update<BM_, BN_, WM_, WN_, true, WPE_>, grid, th, 0, s, a, a.gtab, a.xtab, mt, nt);       \
    else                                                                                                       \
      launch(k_block_update<BM_, BN_, WM_, WN_, false, WPE_>, grid, th, 0, s, a, a.gtab, a.xtab, mt, nt);      \
  } while (0)
  const int R = a.K1 * a.SG * a.B;
  if (a.Mrows % 256 == 0 && R >= 256 && tiles(256, 256) >= 512)
    HAV_BU(256, 256, 128, 64, 2);
  else if (tiles(128, 128) >= 256)
    HAV_BU(128, 128, 64, 64, 3);
  else
    HAV_BU(64, 64, 32, 32, 4);
#undef HAV_BU
}

// ------------------------------------------------------------ Gram blocks past 32 samples
// gram[ks][b][p][k][k2][s][s2] = X[idx_(b,k,p,s)] . X[idx_(b,k2,p,s2)] over
// feature split ks for k2 < k (rows and columns past B zero): per learner and
// block, the 128 x 128 tiles of the rows' Gram matrix (row k*Bp + s) that hold
// such a pair, as two f16 parts of the rows (their magnitude is known).
// 64 learners, 4 blocks of 8 x 64 samples of 3072 features: 0.86 ms.
constexpr int kGB = 128;
__host__ __device__ inline bool gram_tile(int R, int Bp, int mt, int nt) {
  return (min(R, kGB * (mt + 1)) - 1) / Bp > kGB * nt / Bp;
}
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) void k_gram_split(
    const float* __restrict__ X, int64_t ldx, int K, const int32_t* __restrict__ idx, float* __restrict__ gram, int P,
    int K1, int K2, int B, int Bp, int KSG, int cps, int ntiles, int xexp) {
  constexpr int ROWS = 2 * kGB, RPP = 128, NP = ROWS / RPP, MI = 2;
  using T = SplitTile<ROWS, 2>;
  __shared__ __attribute__((aligned(16))) char lds[3][T::kBytes];
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  int t = bid % ntiles;
  const int ks = bid / ntiles % KSG;
  const int pb = bid / (ntiles * KSG), p = pb % P, b = pb / P;
  const int R = K1 * Bp;
  int mt = 0, nt = 0;
  for (;; ) {  // the t-th tile that holds a pair
    if (gram_tile(R, Bp, mt, nt) && t-- == 0) break;
    if (++nt > mt) {
      nt = 0;
      ++mt;
    }
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, lhi = lane >> 5;
  const int wm = (wave >> 2) * 64, wn = (wave & 3) * 32;
  const int c0 = ks * cps, c1 = min(K / kKC, c0 + cps), ns = 4 * (c1 - c0);
  const int sr = tid >> 2, sq = tid & 3;
  const float* src[NP];
  bool ok[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const int r = (i == 0 ? mt : nt) * kGB + sr, k = min(r, R - 1) / Bp, s = min(r, R - 1) - k * Bp;
    ok[i] = r < R && s < B;
    src[i] = X + (int64_t)idx[((int64_t)(b * K1 + k) * P + p) * B + (ok[i] ? s : 0)] * ldx + 4 * sq + (int64_t)c0 * kKC;
  }
  f32x4 v[NP];
  auto load = [&](int s) {
    const int o = 16 * min(s, ns - 1);
#pragma unroll
    for (int i = 0; i < NP; ++i) v[i] = *(const f32x4*)(src[i] + o);
  };
  auto store = [&](char* tile) {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      f32x4 x;
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = ok[i] ? __builtin_amdgcn_ldexpf(v[i][e], xexp) : 0.0f;
      T::put4(tile, sr + RPP * i, sq, x);
    }
  };
  SplitAcc<MI, 1, false> acc;
  acc.clear();
  split_loop8<ROWS, 2>(lds[0], ns, wm, kGB + wn, l32, lhi, wave >> 2, acc, load, store);
  const int n = nt * kGB + wn + l32, k2 = n / Bp, s2 = n - k2 * Bp;
  float* out = gram + (((int64_t)ks * K2 + b) * P + p) * K1 * K1 * Bp * Bp;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = mt * kGB + wm + 32 * i + 8 * (r >> 2) + 4 * lhi + (r & 3), k = m / Bp;
      if (m < R && n < R && k2 < k)
        out[((int64_t)(k * K1 + k2) * Bp + (m - k * Bp)) * Bp + s2] =
            __builtin_amdgcn_ldexpf(acc.sum[i][0][r], -2 * xexp);
    }
}

static int gram_tiles(int K1, int Bp) {
  const int R = K1 * Bp, mts = (R + kGB - 1) / kGB;
  int n = 0;
  for (int mt = 0; mt < mts; ++mt)
    for (int nt = 0; nt <= mt; ++nt) n += gram_tile(R, Bp, mt, nt) ? 1 : 0;
  return n;
}

int gram_split_splits(int P, int K1, int K2, int Bp, int K) {
  // about two workgroups per CU, at least two 64-wide chunks per split
  const int64_t wgs = (int64_t)P * K2 * std::max(1, gram_tiles(K1, Bp));
  const int nch = K / kKC;
  int ks = (int)std::max<int64_t>(1, std::min<int64_t>((512 + wgs - 1) / wgs, nch / 2));
  const int c = (nch + ks - 1) / ks;
  return (nch + c - 1) / c;
}

void launch_gram_split(hipStream_t s, const float* X, int64_t ldx, int K, const int32_t* idx, float* gram, int P,
                       int K1, int K2, int B, int Bp, int KSG, int xexp) {
  const int nt = gram_tiles(K1, Bp), nch = K / kKC;
  if (nt == 0) return;
  launch(k_gram_split, (unsigned)((int64_t)P * K2 * nt * KSG), 512, 0, s, X, ldx, K, idx, gram, P, K1, K2, B, Bp, KSG,
         (nch + KSG - 1) / KSG, nt, xexp);
}

}  // namespace hav
