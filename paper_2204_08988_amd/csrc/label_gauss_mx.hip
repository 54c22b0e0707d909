// Gaussian cluster draw and log-likelihoods in FP32 on the FP32 matrix cores
// (score_mx.hpp): Sec. 4.1 step (e), eq. sample_labels, for d from
// MX_MIN_D to 128.
//
// A wave holds 64 rows in registers and walks the clusters; the records are
// copied to LDS by LDS DMA, all of them once per workgroup while they fit,
// else in groups through two buffers, the next group in flight while the
// current one is scored.  The vector-ALU kernels read a record with scalar
// loads instead: at d = 128 a record of 33 KB does not stay in the 16 KB scalar
// cache, and the draw ran at 11% of the vector ALUs' rate.
//
// Every score has the bits of the vector-ALU form (a log-likelihood of a row with an
// infinite coordinate too), and the draw is the argmax of l_k + g_k (the smaller k on
// ties), so the labels are those of that form.
//
// Bound by the FP32 matrix cores and the vector ALUs together: on this chip the
// two do not overlap (four MFMAs 147 cycles, with 16 vector FMAs 200, at two
// waves per SIMD; the log-likelihoods of larger d run at one).  Measured against the vector-ALU kernels that this one
// replaced: d = 128, N = 1e6, K = 32: 61.9 -> 5.6 ms (9 -> 97 TFLOP/s of
// algorithmic work, 120 executed); d = 100, N = 1e5, K = 32: 15.2 -> 0.56 ms;
// log-likelihoods at d = 32, N = 1e5, K = 20: 1.89 -> 0.15 ms.
#include <algorithm>

#include "kernels.hpp"
#include "score.hpp"
#include "score_mx.hpp"

namespace dpmm {

namespace {

using namespace score;

constexpr int MX_BLOCK = 256;

// the wave's rows [base, base + rows) of x (row 0 read in the place of the others)
template <int RB>
__device__ __forceinline__ void load_chunk(const float* __restrict__ x, long long base, int rows, int d,
                                           float (&xv)[4][4 * RB]) {
  const float* xr[4];
  bool ok[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int r = 16 * t + (threadIdx.x & 15);
    ok[t] = r < rows;
    xr[t] = x + (ok[t] ? (size_t)(base + r) * d : 0);
  }
  mx::load_rows<RB>(xr, ok, d, xv);
}

// Block b labels the points [b per_block, (b + 1) per_block), writes its
// histogram of z.  cg: records per LDS buffer; one
// buffer when it holds all K.
template <int RB>
__global__ __launch_bounds__(MX_BLOCK, 2) void k_label_gauss_mx(const float* __restrict__ x, long long n, int d,
                                                                long long per_block, const float* __restrict__ packed,
                                                                int K, int cg, uint32_t t, uint64_t seed,
                                                                int* __restrict__ z, int* __restrict__ hist) {
  extern __shared__ __align__(16) float smem[];
  const int S = gauss_rec_stride(d);
  const bool single = cg >= K;
  float* buf0 = smem;
  float* buf1 = single ? smem : smem + cg * S;
  int* h = reinterpret_cast<int*>(smem + (single ? 1 : 2) * cg * S + mx::REC_PAD);
  for (int k = threadIdx.x; k < K; k += MX_BLOCK) h[k] = 0;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long long begin = (long long)blockIdx.x * per_block;
  const long long end = begin + per_block < n ? begin + per_block : n;
  const int c0 = cg < K ? cg : K;
  if (begin < end) mx::stage<MX_BLOCK>(buf0, packed, c0 * S);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  bool odd = false;  // which buffer holds the current group
  for (long long chunk = begin; chunk < end; chunk += MX_BLOCK) {
    const long long base = chunk + wave * 64;
    const int rows = (int)(end - base < 64 ? (end - base > 0 ? end - base : 0) : 64);
    float xv[4][4 * RB];
    load_chunk<RB>(x, base, rows, d, xv);
    const uint32_t i = (uint32_t)(base + lane);
    StreamDraw dr;
    dr.init();
    for (int g0 = 0; g0 < K; g0 += cg) {
      const int nk = K - g0 < cg ? K - g0 : cg;
      if (!single) {  // the next group (the first again for the next rows) into the other buffer
        const bool wrap = g0 + cg >= K;
        const int gn = wrap ? 0 : g0 + cg;
        if (!wrap || chunk + MX_BLOCK < end)
          mx::stage<MX_BLOCK>(odd ? buf0 : buf1, packed + (size_t)gn * S, (K - gn < cg ? K - gn : cg) * S);
      }
      mx::lds_cfloat* rec = (mx::lds_cfloat*)(odd ? buf1 : buf0);
      for (int c = 0; c < nk; ++c, rec += S) {
        float q;
        const float cst = rec[0];
        const float fl = dr.floor();
        // a cluster whose partial norm puts it out of range for all 64 points is left
        const bool full = mx::sq_norm<RB>(rec, d, xv, q, [&](float qp) {
          return __ballot(fmaf(-0.5f, qp, cst) > fl) != 0ull;
        });
        if (full) dr.push(fmaf(-0.5f, q, cst), g0 + c, i, t, seed);
      }
      if (!single) {
        __builtin_amdgcn_s_waitcnt(0);  // this wave's part of the next group has landed
        __syncthreads();                // every wave's has, and all are done with the current one
        odd = !odd;
      }
    }
    const int zi = dr.finish(i, t, seed);
    if (lane < rows) {
      z[base + lane] = zi;
      atomicAdd(&h[zi], 1);
    }
  }
  __syncthreads();
  for (int k = threadIdx.x; k < K; k += MX_BLOCK) {
    hist[(size_t)blockIdx.x * K + k] = h[k];
  }
}

// All 3K weighted log-likelihoods of the rows (component j < K: cluster j; K +
// 2 k + h: its sub-clusters), a workgroup taking 256 rows and `jper` components
// (blockIdx.y) at a time: the components are split where the rows alone would
// leave CUs idle.  Sixteen components of a row are gathered in LDS and written
// together (64 bytes of a row at a time instead of 4).
constexpr int LL_GRP = 16;

template <int RB>
__global__ __launch_bounds__(MX_BLOCK, 2) void k_loglik_gauss_mx(const float* __restrict__ x, long long n, int d,
                                                                 const float* __restrict__ packed, int K, int k_max,
                                                                 int cg, int jper, float* __restrict__ out) {
  extern __shared__ __align__(16) float smem[];
  const int S = gauss_rec_stride(d), J = 3 * K;
  const int jb = blockIdx.y * jper, je = jb + jper < J ? jb + jper : J;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float* buf0 = smem;
  float* buf1 = smem + cg * S;
  float* tile = smem + 2 * cg * S + mx::REC_PAD + wave * 64 * (LL_GRP + 1);  // [64][LL_GRP + 1]
  // components [j0, j0 + nj) into dst: the clusters' records, then the sub-clusters'
  auto fetch = [&](float* dst, int j0, int nj) {
    const int a = j0 < K ? (K - j0 < nj ? K - j0 : nj) : 0;
    if (a) mx::stage<MX_BLOCK>(dst, packed + (size_t)j0 * S, a * S);
    if (nj > a) mx::stage<MX_BLOCK>(dst + (size_t)a * S, packed + (size_t)(k_max + j0 + a - K) * S, (nj - a) * S);
  };
  const long long step = (long long)gridDim.x * MX_BLOCK;
  long long chunk = (long long)blockIdx.x * MX_BLOCK;
  if (chunk < n && jb < je) fetch(buf0, jb, je - jb < cg ? je - jb : cg);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  bool odd = false;
  for (; chunk < n; chunk += step) {
    const long long base = chunk + wave * 64;
    const int rows = (int)(n - base < 64 ? (n - base > 0 ? n - base : 0) : 64);
    float xv[4][4 * RB];
    load_chunk<RB>(x, base, rows, d, xv);
    float q = 0.0f;
    for (int g0 = jb; g0 < je; g0 += cg) {
      const int nj = je - g0 < cg ? je - g0 : cg;
      const bool wrap = g0 + cg >= je;
      const int gn = wrap ? jb : g0 + cg;
      if (!wrap || chunk + step < n) fetch(odd ? buf0 : buf1, gn, je - gn < cg ? je - gn : cg);
      mx::lds_cfloat* rec = (mx::lds_cfloat*)(odd ? buf1 : buf0);
      for (int c = 0; c < nj; ++c, rec += S) {
        mx::sq_norm<RB>(rec, d, xv, q, mx::Always());
        const int j = g0 + c, o = j % LL_GRP;
        tile[lane * (LL_GRP + 1) + o] = fmaf(-0.5f, q, rec[0]);
        if (o == LL_GRP - 1 || j == je - 1) {
          const int w = o + 1, j1 = j - o;
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
          for (int e = lane; e < rows * LL_GRP; e += 64) {
            const int r = e / LL_GRP, v = e % LL_GRP;
            if (v < w) out[(size_t)(base + r) * J + j1 + v] = tile[r * (LL_GRP + 1) + v];
          }
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
      }
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      odd = !odd;
    }
    // a score that is not a number (the last stands for all: an infinity meets the zeros above every W's
    // diagonal): where the row has an infinity, again by the plain chain (the stores above have landed)
    if (__ballot(q != q)) {
      const float* xr = x + (size_t)(base + (lane < rows ? lane : 0)) * d;
      bool mine = false;
      for (int c = 0; c < d; ++c) mine = mine || __builtin_isinf(xr[c]);
      if (mine && lane < rows)
        for (int j = jb; j < je; ++j) {
          const float* rec = packed + (size_t)(j < K ? j : k_max + j - K) * S;
          out[(size_t)(base + lane) * J + j] = fmaf(-0.5f, mx::sq_norm_row(rec, d, xr), rec[0]);
        }
    }
  }
}

// staged records of a draw: two workgroups per CU.  (The log-likelihoods' output tile
// comes on top: from d = 29 or so on, wherever the groups are the widest, one per CU)
constexpr size_t MX_LDS_RECORDS = 72 * 1024;
constexpr int MX_LDS_MAX = 160 * 1024;

}  // namespace

hipError_t launch_label_gauss_mx(int d, const float* x, long long n, int G, long long per_block, const float* packed,
                                 int K, uint32_t t, uint64_t seed, int* z, int* hist, hipStream_t s) {
  const size_t rec = (size_t)gauss_rec_stride(d) * sizeof(float);
  int cg = K, bufs = 1;
  if (rec * K > MX_LDS_RECORDS) {
    cg = (int)(MX_LDS_RECORDS / 2 / rec);
    bufs = 2;
  }
  const size_t lds = rec * cg * bufs + mx::REC_PAD * sizeof(float) + (size_t)K * sizeof(int);
  static bool attr_set = false;
  if (!attr_set) {
    const void* fns[7] = {(const void*)k_label_gauss_mx<2>, (const void*)k_label_gauss_mx<3>,
                          (const void*)k_label_gauss_mx<4>, (const void*)k_label_gauss_mx<5>,
                          (const void*)k_label_gauss_mx<6>, (const void*)k_label_gauss_mx<7>,
                          (const void*)k_label_gauss_mx<8>};
    for (const void* f : fns) {
      const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, MX_LDS_MAX);
      if (e != hipSuccess) return e;
    }
    attr_set = true;
  }
  static_assert(mx::row_blocks(MX_MIN_D) == 2, "the smallest form");
#define DPMM_MX_CASE(RB)                                                                                          \
  case RB:                                                                                                        \
    hipLaunchKernelGGL(k_label_gauss_mx<RB>, dim3(G), dim3(MX_BLOCK), lds, s, x, n, d, per_block, packed, K, cg, t, \
                       seed, z, hist);                                                                       \
    break;
  switch (mx::row_blocks(d)) {
    DPMM_MX_CASE(2)
    DPMM_MX_CASE(3)
    DPMM_MX_CASE(4)
    DPMM_MX_CASE(5)
    DPMM_MX_CASE(6)
    DPMM_MX_CASE(7)
    DPMM_MX_CASE(8)
    default:
      return hipErrorInvalidValue;
  }
#undef DPMM_MX_CASE
  return hipGetLastError();
}

hipError_t launch_loglik_gauss(int d, const float* x, long long n, const float* packed, int K, int k_max,
                               float* out, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const size_t rec = (size_t)gauss_rec_stride(d) * sizeof(float);
  int cg = (int)(MX_LDS_RECORDS / 2 / rec);
  // about 2048 workgroups: the components in groups of whole LL_GRPs where n is small
  const int J = 3 * K, grps = (J + LL_GRP - 1) / LL_GRP;
  long long g = (n + MX_BLOCK - 1) / MX_BLOCK;
  if (g > 4096) g = 4096;
  const int ny = (int)std::min<long long>(grps, std::max<long long>(1, 2048 / g));
  const int jper = (grps + ny - 1) / ny * LL_GRP;
  if (cg > jper) cg = jper;
  const size_t lds = rec * cg * 2 + mx::REC_PAD * sizeof(float) + (size_t)MX_BLOCK * (LL_GRP + 1) * sizeof(float);
  static bool attr_set = false;
  if (!attr_set) {
    const void* fns[8] = {(const void*)k_loglik_gauss_mx<1>, (const void*)k_loglik_gauss_mx<2>,
                          (const void*)k_loglik_gauss_mx<3>, (const void*)k_loglik_gauss_mx<4>,
                          (const void*)k_loglik_gauss_mx<5>, (const void*)k_loglik_gauss_mx<6>,
                          (const void*)k_loglik_gauss_mx<7>, (const void*)k_loglik_gauss_mx<8>};
    for (const void* f : fns) {
      const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, MX_LDS_MAX);
      if (e != hipSuccess) return e;
    }
    attr_set = true;
  }
#define DPMM_MX_CASE(RB)                                                                                         \
  case RB:                                                                                                       \
    hipLaunchKernelGGL(k_loglik_gauss_mx<RB>, dim3((unsigned)g, (J + jper - 1) / jper), dim3(MX_BLOCK), lds, s, x, n, \
                       d, packed, K, k_max, cg, jper, out);                                                      \
    break;
  switch (mx::row_blocks(d)) {
    DPMM_MX_CASE(1)
    DPMM_MX_CASE(2)
    DPMM_MX_CASE(3)
    DPMM_MX_CASE(4)
    DPMM_MX_CASE(5)
    DPMM_MX_CASE(6)
    DPMM_MX_CASE(7)
    DPMM_MX_CASE(8)
    default:
      return hipErrorInvalidValue;
  }
#undef DPMM_MX_CASE
  return hipGetLastError();
}

}  // namespace dpmm
