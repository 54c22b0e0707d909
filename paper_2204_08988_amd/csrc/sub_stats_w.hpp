// Sub-labels and statistics of cluster-sorted rows for d <= 32, one kernel per
// dimension (sorted.hip holds the launch of d = 8, 16, 32, sub_stats_any.hip of
// the other dimensions).
#pragma once
#include "kernels.hpp"
#include "score.hpp"

namespace dpmm {

namespace subw {

using score::BLOCK;
using score::score_rec;
typedef __attribute__((__vector_size__(4 * sizeof(double)))) double f64x4;

// Wave-independent kernel for D up to 32: each wave walks its own
// contiguous range of sorted rows in chunks of 64 (one row per lane), with no
// workgroup barriers.  Per chunk:
//   (1) sub-cluster scores: for each run of lanes with the same cluster (rows
//       are sorted by z, so a cluster is a run of lanes) every lane scores the
//       run's two sub-cluster records; control flow stays wave-uniform, so the
//       records are read with scalar loads, and each lane keeps the result of
//       its own run;
//   (2) each row is stored to LDS at its segment-sorted slot: within a run the
//       left rows first, then the right rows;
//   (3) per segment, four rows at a time, v_mfma_f64_16x16x4_f64 adds the
//       16x16 blocks (I <= J) of sum x x^T (dimensions padded to a multiple
//       of 16 with zeros); the same operands give sum x.
// The current cluster's two segments are carried across chunks and flushed
// with global atomics when the cluster changes or the range ends.
template <int D, bool SAMPLE>
__global__ __launch_bounds__(BLOCK) void k_sub_stats_w(const float* __restrict__ x, long long npts, long long n_sorted,
                                                       long long rows_per_wave, const int* __restrict__ perm,
                                                       const int* __restrict__ z, const int* __restrict__ zrow,
                                                       unsigned char* __restrict__ zsub,
                                                       const float* __restrict__ packed, int K, int k_max, uint32_t t,
                                                       uint64_t seed, long long* __restrict__ counts,
                                                       double* __restrict__ moments, const int* __restrict__ cstart,
                                                       const int* __restrict__ ctot, int kbase,
                                                       double* __restrict__ part) {
  constexpr int NB = (D + 15) / 16;  // 16-wide blocks of dimensions
  constexpr int NBLK = NB * (NB + 1) / 2;
  constexpr int LDW = D + 1;  // odd row stride
  constexpr int S = (4 + D + D * (D + 1) / 2 + 3) & ~3;
  constexpr int E = D + D * (D + 1) / 2;
  extern __shared__ float lds[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float* xs = lds + wave * 64 * LDW;
  const unsigned long long below = (1ull << lane) - 1ull;
  const int col = lane & 15;
  f64x4 cL[NBLK], cR[NBLK];
  double sL[NB], sR[NB];
  long long nL = 0, nR = 0;
  int cur_k = -1;
  auto zero_acc = [&]() {
#pragma unroll
    for (int b = 0; b < NBLK; ++b) cL[b] = cR[b] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int b = 0; b < NB; ++b) sL[b] = sR[b] = 0.0;
    nL = nR = 0;
  };
  const long long gw = (long long)blockIdx.x * (BLOCK / 64) + wave;
  const long long w_begin = gw * rows_per_wave;
  const long long w_end = w_begin + rows_per_wave < n_sorted ? w_begin + rows_per_wave : n_sorted;
  int k_first = -1;  // cluster of the wave's first row (partial-slot mode)
  // lane l holds element j of block (I, J) at row 16 I + l / 16 + 4 j, column 16 J + l % 16.
  // Atomic mode (part == nullptr): added to counts[seg], moments[seg].  Slot mode:
  // stored to M (moments layout) and *cnt_out, either the final arrays (the
  // cluster lies in this wave's rows) or a partial slot that k_sub_stats_fix sums.
  auto flush_one = [&](f64x4 (&c)[NBLK], double (&sx)[NB], long long cnt, double* M, long long* cnt_out,
                       double* cnt_d, bool atomic) {
    int blk = 0;
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int J = I; J < NB; ++J, ++blk)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int a = 16 * I + (lane >> 4) + 4 * j, b = 16 * J + col;
          if (a <= b && b < D) {
            double* dst = &M[D + a * D - (a * (a - 1)) / 2 + (b - a)];
            if (atomic)
              atomicAdd(dst, c[blk][j]);
            else
              *dst = c[blk][j];
          }
        }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      double v = sx[b];
      v += __shfl_xor(v, 16);
      v += __shfl_xor(v, 32);
      if (lane < 16 && 16 * b + lane < D) {
        if (atomic)
          atomicAdd(&M[16 * b + lane], v);
        else
          M[16 * b + lane] = v;
      }
    }
    if (lane == 0) {
      if (atomic)
        atomicAdd((unsigned long long*)cnt_out, (unsigned long long)cnt);
      else if (cnt_out)
        *cnt_out = cnt;
      else
        *cnt_d = (double)cnt;
    }
  };
  auto flush = [&]() {
    if (cur_k < 0) return;
    if (!part) {
      if (nL) flush_one(cL, sL, nL, moments + (size_t)(2 * cur_k) * E, &counts[2 * cur_k], nullptr, true);
      if (nR) flush_one(cR, sR, nR, moments + (size_t)(2 * cur_k + 1) * E, &counts[2 * cur_k + 1], nullptr, true);
      return;
    }
    const long long cs = cstart[cur_k - kbase], ce = cs + ctot[cur_k - kbase];
    if (cs >= w_begin && ce <= w_end) {
      // the whole cluster is this wave's: final values, both segments
      flush_one(cL, sL, nL, moments + (size_t)(2 * cur_k) * E, &counts[2 * cur_k], nullptr, false);
      flush_one(cR, sR, nR, moments + (size_t)(2 * cur_k + 1) * E, &counts[2 * cur_k + 1], nullptr, false);
    } else {
      // slot 2 gw: the wave's first cluster; 2 gw + 1: its last (when different); each [2][1 + E]
      double* P = part + (size_t)(2 * gw + (cur_k == k_first ? 0 : 1)) * 2 * (E + 1);
      flush_one(cL, sL, nL, P + 1, nullptr, P, false);
      flush_one(cR, sR, nR, P + (E + 1) + 1, nullptr, P + (E + 1), false);
    }
  };
  // rows [s0, e0) of the wave's LDS tile, four at a time: A = B = the rows' block of dimensions
  auto mfma_rows = [&](f64x4 (&c)[NBLK], double (&sx)[NB], int s0, int e0) {
    for (int g = s0; g < e0; g += 4) {
      // unconditional LDS reads of an element inside the tile (row s0, column 0 for a
      // lane past the rows or the dimensions), then zeroed: no branches, so the reads
      // of the next step can overlap the matrix-core work of this one
      const int rr = g + (lane >> 4);
      const bool ok = rr < e0;
      const int rs = ok ? rr : s0;
      double a[NB];
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const int cc = 16 * b + col;
        const float v = xs[rs * LDW + (cc < D ? cc : 0)];
        a[b] = (ok && cc < D) ? (double)v : 0.0;
      }
#pragma unroll
      for (int b = 0; b < NB; ++b) sx[b] += a[b];
      int blk = 0;
#pragma unroll
      for (int I = 0; I < NB; ++I)
#pragma unroll
        for (int J = I; J < NB; ++J, ++blk) c[blk] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[I], a[J], c[blk], 0, 0, 0);
    }
  };
  zero_acc();
  for (long long c0 = w_begin; c0 < w_end; c0 += 64) {
    const long long r = c0 + lane;
    bool valid = r < w_end;
    long long i = 0;
    int k = -1;
    float xv[D];
    if (valid) {
      i = perm[r];
      // a label outside [0, K) leaves its row out (and never reaches memory)
      valid = (unsigned long long)i < (unsigned long long)npts;
      if (valid) k = zrow ? zrow[r] : z[i];
      valid = valid && (unsigned)k < (unsigned)K;
    }
    if (valid) {
#pragma unroll
      for (int j = 0; j < D; ++j) xv[j] = x[i * D + j];
    } else {
      i = 0;
#pragma unroll
      for (int j = 0; j < D; ++j) xv[j] = 0.0f;
    }
    // ---- (1) sub-labels
    int zs = 0;
    if (SAMPLE) {
      float delta = 0.0f;
      unsigned long long pend = __ballot(valid);
      while (pend) {
        const int lane0 = __ffsll((long long)pend) - 1;
        const int kk = __builtin_amdgcn_readlane(k, lane0);
        const bool mine = valid && k == kk;
        const float* ps = packed + (size_t)(k_max + 2 * kk) * S;
        const float dl = score_rec<D>(ps, xv) - score_rec<D>(ps + S, xv);
        if (mine) delta = dl;
        pend &= ~__ballot(mine);
      }
      if (valid) {
        zs = sub_label_draw(delta, seed, t, (uint32_t)i, K);
        zsub[i] = (unsigned char)zs;
      }
    } else if (valid) {
      zs = zsub[i] ? 1 : 0;
    }
    // ---- (2) segment-sorted slot of each row
    const unsigned long long right = __ballot(valid && zs == 1);
    int pos = 0;
    unsigned long long rem = __ballot(valid);
    while (rem) {
      const int lane0 = __ffsll((long long)rem) - 1;
      const int kk = __builtin_amdgcn_readlane(k, lane0);
      const bool mine = valid && k == kk;
      const unsigned long long mk = __ballot(mine);
      const unsigned long long mR = mk & right, mL = mk & ~right;
      if (mine) pos = lane0 + (zs ? __popcll(mL) + __popcll(mR & below) : __popcll(mL & below));
      rem &= ~mk;
    }
    // the previous chunk's reads of xs are done: same wave, in order
    __builtin_amdgcn_wave_barrier();
    if (valid) {
#pragma unroll
      for (int j = 0; j < D; ++j) xs[pos * LDW + j] = xv[j];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // ---- (3) each run's two segments into the running sums
    rem = __ballot(valid);
    while (rem) {
      const int lane0 = __ffsll((long long)rem) - 1;
      const int kk = __builtin_amdgcn_readlane(k, lane0);
      const unsigned long long mk = __ballot(valid && k == kk);
      if (kk != cur_k) {
        flush();
        zero_acc();
        if (cur_k < 0) k_first = kk;
        cur_k = kk;
      }
      const int cl = __popcll(mk & ~right), cr = __popcll(mk & right);
      nL += cl;
      nR += cr;
      mfma_rows(cL, sL, lane0, lane0 + cl);
      mfma_rows(cR, sR, lane0 + cl, lane0 + cl + cr);
      rem &= ~mk;
    }
  }
  flush();
}

}  // namespace subw

}  // namespace dpmm
