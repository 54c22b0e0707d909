// Sub-labels of cluster-sorted rows from d = 32 on, sub-labels and statistics of the
// smaller dimensions without a launch of their own in sorted.hip: Sec. 4.1 step (f) and
// Sec. 4.4.
//
//   d <= 31   k_sub_stats_w, one instantiation per dimension (the generic
//             kernel before it read both operands of every FMA from LDS:
//             N = 5e5, K = 16: d = 6 551 -> 30 us, 20 742 -> 61, 31 1035 -> 120);
//   d >= 32   k_sub_labels_mx: the two sub-cluster scores of a row on the
//             FP32 matrix cores (score_mx.hpp), with the bits of the
//             vector-ALU form (d = 64, 128 with BF16 tables: on the rows that the bf16x3
//             pass leaves).  The statistics follow in k_sub_stats_w (d = 32) or
//             k_sub_stats_big.
#include "kernels.hpp"
#include "score.hpp"
#include "score_mx.hpp"
#include "sub_stats_w.hpp"

namespace dpmm {

namespace {

constexpr int SLX_BLOCK = 256;

// A workgroup walks a contiguous range of sorted rows, 256 at a time; the two
// records of the current cluster are staged in LDS whenever the cluster changes
// (rows are sorted, so a range holds few; the clusters of the chunk's rows are
// kept in LDS to find the next), and a wave scores its 64 rows if any of them has
// that cluster.  Bound by the matrix cores and the vector ALUs together, as the
// cluster draw; two of its K + 2 evaluations per point.
//
// CORR (d = 32, 64, 128): the rows are centred once, on mu_0, and sub-cluster 1 starts
// its chains at W_1 (mu_0 - mu_1).  With n_dev the rows are the list of n_dev[0] rows
// that the bf16x3 pass left undecided (n_sorted then only bounds the grid).
// N = 1e6: d = 32 62 -> 53 us, d = 64 141, d = 128 452 -> 410 (of 302 at the matrix and
// vector instructions' own rate; the next rows read ahead with one wave per SIMD: 431).
template <int RB, bool CORR>
__global__ __launch_bounds__(SLX_BLOCK, CORR && RB <= 4 ? (RB <= 2 ? 4 : 3) : 2) void k_sub_labels_mx(
    const float* __restrict__ x, int dim, long long n_sorted, long long per_block, const int* __restrict__ perm,
    const int* __restrict__ z, const int* __restrict__ zrow, unsigned char* __restrict__ zsub,
    const float* __restrict__ packed, int K, int k_max, uint32_t t, uint64_t seed, const int* __restrict__ n_dev) {
  extern __shared__ __align__(16) float s_rec[];  // the two records, REC_PAD floats, CORR: [3][d]
  __shared__ int s_k[SLX_BLOCK];                  // clusters of the chunk's rows
  const int d = CORR ? 16 * RB : dim;
  const int S = gauss_rec_stride(d);
  float* s_y0 = s_rec + 2 * S + mx::REC_PAD;  // CORR: zeros, W_1 (mu_0 - mu_1), mu_0 - mu_1
  if (n_dev) {  // the list split evenly over the grid
    n_sorted = *n_dev;
    per_block = ((n_sorted + gridDim.x - 1) / gridDim.x + 63) / 64 * 64;
  }
  const int lane = threadIdx.x & 63, c = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long long begin = (long long)blockIdx.x * per_block;
  const long long end = begin + per_block < n_sorted ? begin + per_block : n_sorted;
  if (CORR && threadIdx.x < d) s_y0[threadIdx.x] = 0.0f;
  int staged = -1;
  for (long long chunk = begin; chunk < end; chunk += SLX_BLOCK) {
    const long long cend = chunk + SLX_BLOCK < end ? chunk + SLX_BLOCK : end;
    const long long mine = chunk + threadIdx.x;
    const int i = mine < cend ? perm[mine] : 0;
    const int k = mine < cend ? (zrow ? zrow[mine] : z[i]) : 0x7fffffff;
    float xv[4][4 * RB];
    const float* xr[4];
    bool ok[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      // row 16 q + c of the wave belongs to lane 16 q + c
      const int r = __shfl(i, 16 * q + c);
      ok[q] = chunk + wave * 64 + 16 * q + c < cend;
      xr[q] = x + (size_t)r * d;
    }
    if (!CORR) mx::load_rows<RB>(xr, ok, d, xv);
    __syncthreads();  // the previous chunk's clusters are read
    s_k[threadIdx.x] = k;
    __syncthreads();
    float delta = 0.0f;
    int cur = __builtin_amdgcn_readfirstlane(s_k[0]);
    for (;;) {
      if (cur != staged) {
        __syncthreads();  // every wave is done with the previous records
        mx::stage<SLX_BLOCK>(s_rec, packed + (size_t)(k_max + 2 * cur) * S, 2 * S);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (CORR) {
          if (threadIdx.x < d) s_y0[2 * d + threadIdx.x] = s_rec[4 + threadIdx.x] - s_rec[S + 4 + threadIdx.x];
          __syncthreads();
          if (threadIdx.x < d) {
            const int r = threadIdx.x;
            const float* w1 = s_rec + S + 4 + d + r * (r + 1) / 2;
            float y = 0.0f;
            // eight reads in flight (those past the row are in the staged records)
            for (int k0 = 0; k0 <= r; k0 += 8) {
              float wv[8], mv[8];
#pragma unroll
              for (int e = 0; e < 8; ++e) {
                wv[e] = w1[k0 + e];
                mv[e] = s_y0[2 * d + k0 + e];
              }
#pragma unroll
              for (int e = 0; e < 8; ++e) y = k0 + e <= r ? fmaf(wv[e], mv[e], y) : y;
            }
            s_y0[d + r] = y;
          }
          __syncthreads();
        }
        staged = cur;
      }
      if (__ballot(k == cur)) {
        mx::lds_cfloat* rec = (mx::lds_cfloat*)s_rec;
        mx::lds_cfloat* y0 = (mx::lds_cfloat*)s_y0;
        if (CORR) {  // centred in place: read again for a wave's next cluster
          mx::load_rows<RB>(xr, ok, d, xv);
#pragma unroll
          for (int s = 0; s < 4 * RB; ++s) {
            const float m = rec[4 + 4 * s + (lane >> 4)];
#pragma unroll
            for (int q = 0; q < 4; ++q) xv[q][s] -= m;
          }
        }
        float sc = 0.0f, dl = 0.0f;
#pragma unroll 1
        for (int sub = 0; sub < 2; ++sub, rec += S, y0 += d) {
          float q;
          if constexpr (CORR)
            q = mx::sq_norm_from<RB>(rec, y0, xv);
          else
            mx::sq_norm<RB>(rec, d, xv, q, mx::Always());
          const float l = fmaf(-0.5f, q, rec[0]);
          dl = sc - l;
          sc = l;
        }
        if (k == cur) delta = dl;
      }
      // the next cluster of the chunk: the smallest above cur (every wave finds the same)
      int nx = 0x7fffffff;
#pragma unroll
      for (int q = 0; q < SLX_BLOCK; q += 64) {
        const int v = s_k[q + lane];
        nx = v > cur && v < nx ? v : nx;
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) nx = min(nx, __shfl_xor(nx, o));
      if (nx == 0x7fffffff) break;
      cur = __builtin_amdgcn_readfirstlane(nx);
    }
    if (mine < cend) zsub[i] = (unsigned char)sub_label_draw(delta, seed, t, (uint32_t)i, K);
  }
}

}  // namespace

hipError_t launch_sub_labels_mx(int d, const float* x, long long n, const int* perm, const int* z, const int* zrow,
                                unsigned char* zsub, const float* packed, int K, int k_max, uint32_t t, uint64_t seed,
                                hipStream_t s, const int* n_dev) {
  if (n == 0) return hipSuccess;
  const bool corr = d == 32 || d == 64 || d == 128;
  const size_t lds = (size_t)(2 * gauss_rec_stride(d) + mx::REC_PAD + (corr ? 3 * d + 8 : 0)) * sizeof(float);
  static bool attr_set = false;
  if (!attr_set) {
    const void* fns[8] = {(const void*)k_sub_labels_mx<3, false>, (const void*)k_sub_labels_mx<4, false>,
                          (const void*)k_sub_labels_mx<5, false>, (const void*)k_sub_labels_mx<6, false>,
                          (const void*)k_sub_labels_mx<7, false>, (const void*)k_sub_labels_mx<8, false>,
                          (const void*)k_sub_labels_mx<4, true>,  (const void*)k_sub_labels_mx<8, true>};
    for (const void* f : fns) {
      const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 80 * 1024);
      if (e != hipSuccess) return e;
    }
    attr_set = true;
  }
  // at most four workgroups per CU (d = 64, 128: the three, two resident at once), each
  // on a range of whole steps (d = 32, 64, 128: whole waves)
  const long long cap = d == 128 ? 512 : (d == 64 ? 768 : 1024), unit = corr ? 64 : SLX_BLOCK;
  long long per = (n + cap - 1) / cap;
  per = (per + unit - 1) / unit * unit;
  const unsigned G = (unsigned)((n + per - 1) / per);
#define DPMM_SLX(RB, CORR)                                                                                            \
  hipLaunchKernelGGL((k_sub_labels_mx<RB, CORR>), dim3(G), dim3(SLX_BLOCK), lds, s, x, d, n, per, perm, z, zrow, zsub, \
                     packed, K, k_max, t, seed, n_dev)
  if (corr) {
    if (d == 32)
      DPMM_SLX(2, true);
    else if (d == 64)
      DPMM_SLX(4, true);
    else
      DPMM_SLX(8, true);
    return hipGetLastError();
  }
  switch (mx::row_blocks(d)) {
    case 3: DPMM_SLX(3, false); break;
    case 4: DPMM_SLX(4, false); break;
    case 5: DPMM_SLX(5, false); break;
    case 6: DPMM_SLX(6, false); break;
    case 7: DPMM_SLX(7, false); break;
    case 8: DPMM_SLX(8, false); break;
    default: return hipErrorInvalidValue;
  }
#undef DPMM_SLX
  return hipGetLastError();
}

hipError_t launch_sub_stats_w_any(int d, bool sample, const float* x, long long npts, long long n, long long rpw,
                                  const int* perm, const int* z, const int* zrow, unsigned char* zsub,
                                  const float* packed, int K, int k_max, uint32_t t, uint64_t seed, long long* counts,
                                  double* moments, const int* cstart, const int* ctot, int kbase, double* part,
                                  hipStream_t s) {
  const long long nw = (n + rpw - 1) / rpw;
  const unsigned grid = (unsigned)((nw + 3) / 4);
  const size_t lds = (size_t)4 * 64 * (d + 1) * sizeof(float);
#define DPMM_ANY(DD, SS)                                                                                              \
  hipLaunchKernelGGL((subw::k_sub_stats_w<DD, SS>), dim3(grid), dim3(score::BLOCK), lds, s, x, npts, n, rpw, perm, z, \
                     zrow, zsub, packed, K, k_max, t, seed, counts, moments, cstart, ctot, kbase, part)
#define DPMM_ANY_CASE(DD)  \
  case DD:                 \
    if (sample)            \
      DPMM_ANY(DD, true);  \
    else                   \
      DPMM_ANY(DD, false); \
    break;
// d <= 4 draws its sub-labels with its labels
#define DPMM_ANY_SMALL(DD)                   \
  case DD:                                   \
    if (sample) return hipErrorInvalidValue; \
    DPMM_ANY(DD, false);                     \
    break;
  switch (d) {
    DPMM_ANY_SMALL(1)
    DPMM_ANY_SMALL(2)
    DPMM_ANY_SMALL(3)
    DPMM_ANY_SMALL(4)
    DPMM_ANY_CASE(5)
    DPMM_ANY_CASE(6)
    DPMM_ANY_CASE(7)
    DPMM_ANY_CASE(9)
    DPMM_ANY_CASE(10)
    DPMM_ANY_CASE(11)
    DPMM_ANY_CASE(12)
    DPMM_ANY_CASE(13)
    DPMM_ANY_CASE(14)
    DPMM_ANY_CASE(15)
    DPMM_ANY_CASE(17)
    DPMM_ANY_CASE(18)
    DPMM_ANY_CASE(19)
    DPMM_ANY_CASE(20)
    DPMM_ANY_CASE(21)
    DPMM_ANY_CASE(22)
    DPMM_ANY_CASE(23)
    DPMM_ANY_CASE(24)
    DPMM_ANY_CASE(25)
    DPMM_ANY_CASE(26)
    DPMM_ANY_CASE(27)
    DPMM_ANY_CASE(28)
    DPMM_ANY_CASE(29)
    DPMM_ANY_CASE(30)
    DPMM_ANY_CASE(31)
    default:
      return hipErrorInvalidValue;
  }
#undef DPMM_ANY_SMALL
#undef DPMM_ANY_CASE
#undef DPMM_ANY
  return hipGetLastError();
}

}  // namespace dpmm
