// FP32 component scores of 64 points per wave on the FP32 matrix cores, bit for
// bit the scores of score_rec (score.hpp).
//
// v_mfma_f32_16x16x4_f32 adds its four products to an accumulator one after the
// other in increasing k, each as a fused multiply-add rounded to FP32 (checked
// against fmaf over 300 000 results with exponents from 2^-70 to 2^70, denormal
// results included).  A chain of these instructions over k is therefore the
// chain y = fma(w[c], dx[c], y), c = 0, 1, ..., of the vector-ALU form, and the
// zeros that pad W above its diagonal and below its last row leave a finite
// chain unchanged (fma(0, dx, y) = y).  Times an infinite dx they give a NaN where
// the chain over c <= r has none: a caller that returns the score takes such a row's
// norm from sq_norm_row; a draw does not tell the two apart (a score of -inf and one
// that is not a number both lose).  The squared norm q = fma(y_r, y_r, q)
// runs over increasing r as there: after the rows of a 16-row block are formed,
// a 4 x 4 transpose over the lane groups (v_permlane32_swap, v_permlane16_swap)
// gives every lane all 16 rows of one point.
//
// Layout: the wave's 64 points are four tiles of 16.  Lane l = 16 g + c holds,
// for point c of every tile t, the coordinates 4 s + g (x[t][s]); it supplies
// W[i][4 s + g], i = c, as the A operand (one LDS read for four tiles) and owns
// point 16 g + c = l of the 64 at the end.
//
// Cost at dimension d: sum over the 16-row blocks of 4 tiles x min(4 (rb + 1),
// d / 4) instructions of 32 cycles: 18 432 cycles per 64 points at d = 128
// (the vector ALUs: 8 384 FMAs = 33 536 cycles), 1 536 at d = 32 (2 368), 512
// at d = 16 (608 to 672).  Blocks of 32 rows (32x32x2) would spend 20 480 and
// 2 048 on the wider diagonal blocks.
#pragma once
#include "common.hpp"

namespace dpmm {
namespace mx {

typedef float f32x4 __attribute__((ext_vector_type(4)));
// floats that may be read past the end of the last staged record (masked)
constexpr int REC_PAD = 16;

__host__ __device__ constexpr int row_blocks(int d) { return (d + 15) / 16; }

typedef __attribute__((address_space(3))) void lds_void;

// Copies `words` floats (a multiple of 4) from src to LDS by LDS DMA, every
// thread of a workgroup of BLK taking part; landed after a wait and a barrier.
template <int BLK>
__device__ __forceinline__ void stage(float* dst, const float* src, int words) {
  const int n4 = words >> 2;
  for (int f0 = 0; f0 < n4; f0 += BLK) {
    const int f = f0 + threadIdx.x;
    if (f < n4)
      __builtin_amdgcn_global_load_lds((const void*)(src + 4 * (size_t)f), (lds_void*)(dst + 4 * (f & ~63)), 16, 0, 0);
  }
}

// Four rows (registers v0 .. v3 of tiles 0 .. 3, row 4 g + r of lane group g)
// transposed: v_j becomes row 4 j + r of the lane's own tile.
__device__ __forceinline__ void transpose4(float& v0, float& v1, float& v2, float& v3) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v0), __float_as_uint(v2), false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v1), __float_as_uint(v3), false, false);
  const auto e = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
  const auto f = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
  v0 = __uint_as_float(e[0]);
  v1 = __uint_as_float(e[1]);
  v2 = __uint_as_float(f[0]);
  v3 = __uint_as_float(f[1]);
}

// a and b: sums over half the coordinates, of point l % 32 of one 32-point tile and of
// the next, the other half of them in lane l ^ 32.  The whole sum of the lane's own point
// (lanes 0-31 the first tile's, 32-63 the second's).
__device__ __forceinline__ float half_sums(float a, float b) {
  const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
}

// x[t][s] of the rows xr[t] (the lane's row 16 t + c of each tile), zero where !ok[t]
// (xr[t] must be readable all the same) and past the dimension.  The four lanes
// of a row read 64 consecutive bytes of it at a time and trade them by
// transpose4; 4-byte loads would touch every line of the row eight times, with
// the wave's 64 rows larger than the L1.  Rows need not be 16-byte aligned.
template <int RB>
__device__ __forceinline__ void load_rows(const float* const (&xr)[4], const bool (&ok)[4], int d,
                                          float (&x)[4][4 * RB]) {
  typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
  const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
#pragma unroll
    for (int j = 0; j < RB; ++j) {
      float v[4];
      if (j < RB - 1 || d == 16 * RB) {
        const f32x4u u = *reinterpret_cast<const f32x4u*>(xr[t] + 16 * j + 4 * g);
        v[0] = u.x, v[1] = u.y, v[2] = u.z, v[3] = u.w;
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int c = 16 * j + 4 * g + q;
          const float u = xr[t][c < d ? c : 0];
          v[q] = c < d ? u : 0.0f;
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) x[t][4 * j + q] = ok[t] ? v[q] : 0.0f;
    }
  }
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int j = 0; j < RB; ++j)
      transpose4(x[t][4 * j], x[t][4 * j + 1], x[t][4 * j + 2], x[t][4 * j + 3]);
}

// Squared norm q of the lane's own point under the record p (in LDS, REC_PAD
// floats readable past it).  `go(q)` is asked after every 16-row block but the
// last whether the wave still needs the rest: q only grows from block to block,
// so the score of the partial norm bounds the full one from above, also in
// rounded arithmetic.  Returns false when it stopped.
//
// The steps of a block are pipelined by hand: W and the mean PF steps ahead of
// their use, x - mu one step ahead, so that neither an LDS read nor the wait
// from a vector instruction to the matrix instruction that reads it stands
// between two matrix instructions.
typedef __attribute__((address_space(3))) const float lds_cfloat;

// `go` of a caller that always wants the whole norm: a branch that the compiler
// cannot fold, so that the row blocks stay separate basic blocks (in one block it
// loads the operands of all of them first and spills)
struct Always {
  __device__ __forceinline__ bool operator()(float) const {
    int one = 1;
    asm volatile("" : "+s"(one));
    return one != 0;
  }
};

template <int RB, typename GoFn>
__device__ __forceinline__ bool sq_norm(lds_cfloat* p, int d, const float (&x)[4][4 * RB], float& q, GoFn go) {
  constexpr int PF = 3;
  const int lane = threadIdx.x & 63, g = lane >> 4, i = lane & 15;
  q = 0.0f;
  const int ext = d - 16 * (RB - 1);  // rows of the last block
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const bool last = rb == RB - 1;
    const int NS = 4 * (rb + 1);
    const int r = 16 * rb + i;
    const bool rok = !last || i < ext;
    const int rr = rok ? r : d - 1;
    lds_cfloat* wr = p + 4 + d + rr * (rr + 1) / 2 + g;
    lds_cfloat* mu = p + 4 + g;
    asm volatile("" : "+v"(mu));  // read again per block, not held across the blocks
    float w[4 * RB], m[4 * RB], b[2][4];
    auto load = [&](int s) __attribute__((always_inline)) {
      w[s] = wr[4 * s];
      m[s] = mu[4 * s];
    };
    // the operands of step s: zero above the diagonal, below the last row and past the dimension
    auto ready = [&](int s) __attribute__((always_inline)) {
      if (s >= 4 * rb) w[s] = 4 * s + g <= r && rok ? w[s] : 0.0f;
      else if (last) w[s] = rok ? w[s] : 0.0f;
      if (last && s >= 4 * rb) m[s] = 4 * s + g < d ? m[s] : 0.0f;
#pragma unroll
      for (int t = 0; t < 4; ++t) b[s & 1][t] = x[t][s] - m[s];
    };
#pragma unroll
    for (int s = 0; s < PF && s < NS; ++s) load(s);
    ready(0);
    f32x4 a[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) a[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 4 * RB; ++s) {
      if (s >= NS) continue;
      if (s + PF < NS) load(s + PF);
      if (s + 1 < NS) ready(s + 1);
      __builtin_amdgcn_sched_barrier(0);
      // the last block's steps past the dimension are skipped (uniform)
      if (!(last && s > 4 * rb) || 4 * (s - 4 * rb) < ext) {
#pragma unroll
        for (int t = 0; t < 4; ++t) a[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[s], b[s & 1][t], a[t], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float y0 = a[0][u], y1 = a[1][u], y2 = a[2][u], y3 = a[3][u];
      transpose4(y0, y1, y2, y3);
      a[0][u] = y0;
      a[1][u] = y1;
      a[2][u] = y2;
      a[3][u] = y3;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int u = 0; u < 4; ++u) q = fmaf(a[j][u], a[j][u], q);
    if (!last && !go(q)) return false;
  }
  return true;
}

// The squared norm of one row by the plain chain, row and record in memory: for rows
// with an infinite coordinate.  Ends at the first row of W that gives a NaN.
__device__ __forceinline__ float sq_norm_row(const float* __restrict__ p, int d, const float* __restrict__ x) {
  const float* w = p + 4 + d;
  float q = 0.0f;
#pragma unroll 1
  for (int r = 0; r < d && q == q; w += ++r) {
    float y = 0.0f;
#pragma unroll 1
    for (int c = 0; c <= r; ++c) y = fmaf(w[c], x[c] - p[4 + c], y);
    q = fmaf(y, y, q);
  }
  return q;
}

// Squared norm of W v + y0 for the rows v = x (already centred; d = 16 RB), W of the
// record p, y0 the d starting values of the chains (y0 in LDS).  The rows' squares
// are summed in two chains, those with bit 2 of the row clear and set, the order of
// 32 x 32 accumulators.
template <int RB>
__device__ __forceinline__ float sq_norm_from(lds_cfloat* p, lds_cfloat* y0, const float (&x)[4][4 * RB]) {
  constexpr int PF = 3, D = 16 * RB;
  typedef __attribute__((address_space(3))) const f32x4 lds_f32x4;
  const int lane = threadIdx.x & 63, g = lane >> 4, i = lane & 15;
  float q0 = 0.0f, q1 = 0.0f;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int NS = 4 * (rb + 1), r = 16 * rb + i;
    lds_cfloat* wr = p + 4 + D + r * (r + 1) / 2 + g;
    const f32x4 start = *(lds_f32x4*)(y0 + 16 * rb + 4 * g);
    float w[4 * RB];
#pragma unroll
    for (int s = 0; s < PF && s < NS; ++s) w[s] = wr[4 * s];
    f32x4 a[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) a[t] = start;
#pragma unroll
    for (int s = 0; s < 4 * RB; ++s) {
      if (s >= NS) continue;
      if (s + PF < NS) w[s + PF] = wr[4 * (s + PF)];
      if (s >= 4 * rb) w[s] = 4 * s + g <= r ? w[s] : 0.0f;  // above the diagonal
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < 4; ++t) a[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[s], x[t][s], a[t], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float v0 = a[0][u], v1 = a[1][u], v2 = a[2][u], v3 = a[3][u];
      transpose4(v0, v1, v2, v3);
      a[0][u] = v0;
      a[1][u] = v1;
      a[2][u] = v2;
      a[3][u] = v3;
    }
#pragma unroll
    for (int j = 0; j < 4; j += 2)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        q0 = fmaf(a[j][u], a[j][u], q0);
        q1 = fmaf(a[j + 1][u], a[j + 1][u], q1);
      }
    if (rb < RB - 1 && !Always()(q0)) break;
  }
  return q0 + q1;
}

}  // namespace mx
}  // namespace dpmm
