// Cluster-sorted second half of the Gaussian label step, for d >= 5:
// Sec. 4.1 step (f) (sub-labels) and the statistics update of Sec. 4.4.
//
// After the cluster draw, points are counting-sorted by z:
//   k_hist_z     per-block histogram of z over contiguous point ranges (only
//                when the label kernel did not produce it);
//   k_scan_hist  per-(block, cluster) output offsets;
//   k_scatter_z  perm[offset] = i, zsort[offset] = z_i (the cluster of each
//                sorted row, read coalesced by the kernels below).
// Then, over the sorted order (a cluster is a run of rows):
//   d <= 31      k_sub_stats_w: sub-labels and statistics in one pass;
//   d = 32       k_sub_labels_mx (sub_stats_any.hip), then k_sub_stats_w;
//   d = 64, 128  k_sub_labels_mx (with BF16 tables behind the bf16x3 pass),
//                then k_sub_stats_big;
//   other d      k_sub_labels_mx, then k_sub_stats_big over rows padded with
//                zero columns to 64 or 128.
// Each walks contiguous ranges of rows, keeps the current cluster's sums and
// leaves those of clusters that span ranges to k_sub_stats_fix.
#include <utility>

#include "kernels.hpp"
#include "score.hpp"
#include "sub_stats_w.hpp"

namespace dpmm {

namespace {

using score::BLOCK;
using subw::k_sub_stats_w;
typedef __attribute__((__vector_size__(4 * sizeof(double)))) double f64x4;

// Inclusive scan over a workgroup of `NT` threads (integer: exact in any
// order), left in buf (NT ints) as well: shuffles within each wave, then the
// preceding waves' totals (staged in buf's first entries); three barriers.
template <int NT>
__device__ __forceinline__ int block_inclusive_scan_n(int v, int* buf) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(v, o);
    if (lane >= o) v += u;
  }
  if (lane == 63) buf[w] = v;
  __syncthreads();
  int add = 0;
#pragma unroll
  for (int q = 0; q < NT / 64; ++q) add += q < w ? buf[q] : 0;
  v += add;
  __syncthreads();  // every wave has read the totals
  buf[tid] = v;
  __syncthreads();
  return v;
}

__device__ __forceinline__ int block_inclusive_scan(int v, int* buf) { return block_inclusive_scan_n<BLOCK>(v, buf); }

}  // namespace

__global__ __launch_bounds__(BLOCK) void k_hist_z(const int* __restrict__ z, long long n, long long per_block, int K,
                                                  int* __restrict__ hist, const int* __restrict__ mode) {
  if (mode && *mode == 0) return;
  extern __shared__ int h[];
  for (int k = threadIdx.x; k < K; k += BLOCK) h[k] = 0;
  __syncthreads();
  const long long begin = (long long)blockIdx.x * per_block;
  const long long end = begin + per_block < n ? begin + per_block : n;
  for (long long i = begin + threadIdx.x; i < end; i += BLOCK) {
    const int zi = z[i];
    if ((unsigned)zi < (unsigned)K) atomicAdd(&h[zi], 1);
  }
  __syncthreads();
  for (int k = threadIdx.x; k < K; k += BLOCK) {
    hist[(size_t)blockIdx.x * K + k] = h[k];
  }
}

// One workgroup per cluster k: offs[b][k] = sum_{b' < b} hist[b'][k] (0 in row 0)
// and the total tot[k].  k_scatter_z adds the clusters' starts.  (The blocks of the
// label kernels and k_hist_z used to add their counts to cleared totals: at N = 1e6,
// K = 16 two thousand atomics on each of sixteen addresses, 24.8 us of k_hist_z
// against 3.5 us now, and a launch to clear them.)
constexpr int SORT_BLOCKS = 2048;  // plan_blocks makes no more
__global__ __launch_bounds__(BLOCK) void k_scan_hist(const int* __restrict__ hist, int G, int K,
                                                     int* __restrict__ tot, int* __restrict__ offs,
                                                     const int* __restrict__ mode) {
  if (mode && *mode == 0) return;
  constexpr int PER = SORT_BLOCKS / BLOCK;
  __shared__ int buf[BLOCK];
  const int k = blockIdx.x, g0 = threadIdx.x * PER;
  int v[PER], local = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) v[j] = g0 + j < G ? hist[(size_t)(g0 + j) * K + k] : 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) local += v[j];
  const int incl = block_inclusive_scan(local, buf);
  int run = incl - local;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    if (g0 + j < G) offs[(size_t)(g0 + j) * K + k] = run;
    run += v[j];
  }
  if (threadIdx.x == BLOCK - 1) tot[k] = incl;
}

// Stable scatter: within block b the rows of a cluster keep their index
// order, so the sorted order (and every float64 sum taken over it) does not
// depend on timing.  Wave w owns the contiguous quarter [begin + w q, begin +
// (w + 1) q) of the block's range (q = per_block / 4, a multiple of 64): it
// counts its rows per cluster (LDS integer atomics, exact), its cursor for
// cluster k is the block's offset plus the counts of the waves before it, and
// it then walks its quarter 64 rows at a time.  The lanes holding the same
// cluster are found with one ballot per bit of the cluster index (the lanes
// that agree with this lane on every bit); a lane's rank among them is the
// count of those below it, and the highest of them moves the cursor.  The
// clusters' starts are the exclusive sums of tot; block 0 leaves them in row 0 of
// offs (whose own offsets are 0) for the kernels that follow.
__global__ __launch_bounds__(BLOCK) void k_scatter_z(const int* __restrict__ z, long long n, long long per_block,
                                                     int K, const int* __restrict__ tot, int* __restrict__ offs,
                                                     int* __restrict__ perm, int* __restrict__ zsort,
                                                     const int* __restrict__ mode) {
  if (mode && *mode == 0) return;
  extern __shared__ int cur[];  // [4][K]
  __shared__ int buf[BLOCK];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int q = threadIdx.x; q < 4 * K; q += BLOCK) cur[q] = 0;
  __syncthreads();
  const long long begin = (long long)blockIdx.x * per_block;
  const long long end = begin + per_block < n ? begin + per_block : n;
  const long long quarter = per_block / 4;
  const long long wb = begin + w * quarter;
  const long long we = wb + quarter < end ? wb + quarter : end;
  int* mine = cur + w * K;
  for (long long i = wb + lane; i < we; i += 64) {
    const int zi = z[i];
    if ((unsigned)zi < (unsigned)K) atomicAdd(&mine[zi], 1);
  }
  // a contiguous share of the clusters per thread
  const int per = (K + BLOCK - 1) / BLOCK;
  const int ka = threadIdx.x * per < K ? threadIdx.x * per : K, kb = ka + per < K ? ka + per : K;
  int local = 0;
  for (int k = ka; k < kb; ++k) local += tot[k];
  int start = block_inclusive_scan(local, buf) - local;  // (its barriers complete the counts above)
  for (int k = ka; k < kb; ++k) {
    int run = start;
    if (blockIdx.x == 0)
      offs[k] = start;
    else
      run += offs[(size_t)blockIdx.x * K + k];
    start += tot[k];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = cur[u * K + k];
      cur[u * K + k] = run;
      run += c;
    }
  }
  __syncthreads();
  const unsigned long long below = (1ull << lane) - 1ull;
  int nbits = 1;
  while ((1 << nbits) < K) ++nbits;
  for (long long c0 = wb; c0 < we; c0 += 64) {
    const long long i = c0 + lane;
    const int zi = i < we ? z[i] : -1;
    const bool v = (unsigned)zi < (unsigned)K;
    unsigned long long m = __ballot(v);
    for (int b = 0; b < nbits; ++b) {
      const unsigned long long on = __ballot(v && ((zi >> b) & 1));
      m &= ((zi >> b) & 1) ? on : ~on;
    }
    int base = 0;
    if (v) base = mine[zi];
    // every lane has read its cursor before any moves (wave order)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (v) {
      const int pos = base + __popcll(m & below);
      perm[pos] = (int)i;
      zsort[pos] = zi;
      if ((m >> lane) == 1ull) mine[zi] = base + __popcll(m);  // the highest lane of its cluster
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// Slot mode of the sorted-order statistics kernels: the counts and moments of
// every cluster whose rows span several row ranges (rpw rows each: a wave of
// k_sub_stats_w, a workgroup of the other kernels) are the sums of those
// ranges' partial slots (2 g for the range's first cluster, 2 g + 1 for its
// last); empty clusters get zeros; a cluster inside one range was written by
// it.  Grid (entries / FIX_EN, clusters): cluster kbase + blockIdx.y, whose
// start and size are cstart / ctot[blockIdx.y].  FIX_PH phases of threads take
// every FIX_PH-th slot of FIX_EN entries, and their sums are added in a fixed
// order (the result does not depend on timing).
constexpr int FIX_PH = 16, FIX_EN = 16;
__global__ __launch_bounds__(FIX_PH * FIX_EN) void k_sub_stats_fix(int E, long long rpw, const int* __restrict__ cstart,
                                                                 const int* __restrict__ ctot,
                                                                 const double* __restrict__ part,
                                                                 long long* __restrict__ counts,
                                                                 double* __restrict__ moments, int kbase) {
  __shared__ double red[FIX_PH][FIX_EN];
  const int k = blockIdx.y;
  const int W = 2 * (E + 1);
  const int el = threadIdx.x % FIX_EN, ph = threadIdx.x / FIX_EN;
  const int e = blockIdx.x * FIX_EN + el;
  const long long cs = cstart[k], cnt = ctot[k];
  const long long ga = cnt > 0 ? cs / rpw : 0, gb = cnt > 0 ? (cs + cnt - 1) / rpw : -1;
  if (cnt > 0 && ga == gb) return;  // written by the range that holds it (uniform over the block)
  double v = 0.0;
  if (e < W) {
#pragma unroll 4
    for (long long g = ga + ph; g <= gb; g += FIX_PH)
      v += part[(size_t)(2 * g + (g == ga && cs != g * rpw ? 1 : 0)) * W + e];
  }
  red[ph][el] = v;
  __syncthreads();
  if (ph != 0 || e >= W) return;
  double sum = 0.0;
  for (int q = 0; q < FIX_PH; ++q) sum += red[q][el];
  const int h = e / (E + 1), f = e - h * (E + 1);
  const size_t seg = 2 * ((size_t)k + kbase) + h;
  if (f == 0)
    counts[seg] = (long long)sum;  // a sum of integer counts below 2^53: exact
  else
    moments[seg * E + (f - 1)] = sum;
}

namespace {

struct SortedPlan {
  int G;
  long long per_block;
};

SortedPlan plan_blocks(long long n, int K, long long hist_cap, int block_rows) {
  long long G = (n + block_rows - 1) / block_rows;
  if (G > SORT_BLOCKS) G = SORT_BLOCKS;
  while (G > 1 && G * K > hist_cap) G = (G + 1) / 2;
  if (G < 1) G = 1;
  long long per = (n + G - 1) / G;
  per = ((per + BLOCK - 1) / BLOCK) * BLOCK;
  G = (n + per - 1) / per;
  if (G < 1) G = 1;
  return SortedPlan{(int)G, per};
}

constexpr int BIG_THREADS = 512;  // 8 waves: 0-3 own the left segment, 4-7 the right
// sorted rows per tile: 64 KB of FP32 rows, so that two tiles fit in LDS
constexpr int big_rows_of(int d) { return 16384 / d; }
typedef __attribute__((address_space(3))) void lds_void;

__device__ __forceinline__ int block_inclusive_scan_big(int v, int* buf) { return block_inclusive_scan_n<BIG_THREADS>(v, buf); }

// Upper 16 x 16 block u (row-major over I <= J) of an NB x NB block grid.
constexpr int blk_i(int u, int nb) {
  int a = 0;
  while (a < nb && u >= nb - a) {
    u -= nb - a;
    ++a;
  }
  return a;
}
constexpr int blk_j(int u, int nb) { return u - (blk_i(u, nb) * nb - blk_i(u, nb) * (blk_i(u, nb) - 1) / 2) + blk_i(u, nb); }

// The accumulator updates of one four-row step for wave quarter WQ: block
// u = WQ + 4 j of accumulator j, its (I, J) fixed at compile time so that the
// operands are plain registers.
template <int U, int NB>
constexpr int BLK_I = blk_i(U, NB) < NB ? blk_i(U, NB) : NB - 1;
template <int U, int NB>
constexpr int BLK_J = blk_i(U, NB) < NB ? blk_j(U, NB) : NB - 1;

template <int NB, int WQ, int TPW, int... J>
__device__ __forceinline__ void big_mfmas(f64x4 (&acc)[TPW], const double (&xv)[NB], std::integer_sequence<int, J...>) {
  constexpr int NT = NB * (NB + 1) / 2;
  ((WQ + 4 * J < NT
        ? (void)(acc[J] = __builtin_amdgcn_mfma_f64_16x16x4f64(xv[BLK_I<WQ + 4 * J, NB>], xv[BLK_J<WQ + 4 * J, NB>],
                                                               acc[J], 0, 0, 0))
        : (void)0),
   ...);
}

// Column held by lane i (of 16) for column block I in the statistics tile:
// lane i reads its D / 16 columns as one contiguous piece of the row (one or
// two 16-byte LDS reads), so block I is the column set {col(I, i)}.  At
// d = 128 the two halves of a lane's piece are read in an order that depends
// on bits 2 and 3 of i, so that any 8 or 16 consecutive lanes reading one row
// hit distinct LDS banks.
template <int D>
__device__ __forceinline__ int big_col(int blk, int i) {
  if constexpr (D == 128) {
    const int s = ((i >> 2) ^ (i >> 3)) & 1;
    return 8 * i + (blk ^ (4 * s));
  } else {
    return 4 * i + blk;
  }
}

// Rows [st, st + cnt) of a tile's order list, four at a time, into the
// accumulators of wave quarter WQ (upper blocks WQ, WQ + 4, ...): each step
// reads the lane's piece of its row once and feeds every block from it (a
// lane past the segment reads the zero row R).  rd0 / rd1: the lane's two
// 16-byte offsets in a row (rd1 unused at d = 64).
template <int D, int WQ, int R, int TPW>
__device__ __forceinline__ void big_rows(f64x4 (&acc)[TPW], double (&sx)[D / 64], const float* __restrict__ xs,
                                         const int* __restrict__ order, int st, int cnt, int lane, int rd0, int rd1) {
  constexpr int NB = D / 16;
  const int p = lane >> 4;
  // (a two-step software pipeline of these reads measured the same: the other
  // wave of the SIMD covers their latency, and while an LDS DMA is in flight
  // the compiler waits for every LDS read before its first use anyway)
  for (int g = 0; g < cnt; g += 4) {
    const int q = g + p;
    const float* rp = xs + (q < cnt ? order[st + q] : R) * D;
    const float4 a = *reinterpret_cast<const float4*>(rp + rd0);
    double xv[NB];
    xv[0] = (double)a.x;
    xv[1] = (double)a.y;
    xv[2] = (double)a.z;
    xv[3] = (double)a.w;
    if constexpr (NB == 8) {
      const float4 b = *reinterpret_cast<const float4*>(rp + rd1);
      xv[4] = (double)b.x;
      xv[5] = (double)b.y;
      xv[6] = (double)b.z;
      xv[7] = (double)b.w;
    }
    big_mfmas<NB, WQ>(acc, xv, std::make_integer_sequence<int, TPW>{});
    // sum x over the quarter's column blocks WQ, WQ + 4, ...: lane l adds
    // column col(block, l % 16) of its row
#pragma unroll
    for (int j = 0; j < D / 64; ++j) sx[j] += xv[WQ + 4 * j];
  }
}

// Statistics for d in {64, 128} over the cluster-sorted order (the sub-labels
// are drawn before, by the sub-label kernels), with sum x x^T on the FP64
// matrix cores.  A workgroup of 8 waves walks a contiguous range of tiles of
// big_rows_of(D) sorted rows (64 KB of rows each), two tiles' rows in LDS:
//   (1) the next tile's rows are copied into the other LDS buffer by LDS DMA
//       (global_load_lds, 16 bytes per lane, no registers) while this tile's
//       matrix-core work runs; its point indices, clusters and sub-labels are
//       loaded into registers at the same time;
//   (2) rows are grouped by segment (run of a cluster, sub-label), each
//       segment keeping the rows' sorted order (ranks from one block scan);
//   (3) per segment, four rows at a time, v_mfma_f64_16x16x4_f64 adds
//       X_I^T X_J to the upper 16 x 16 blocks (I, J) of sum x x^T (column
//       blocks as big_col gives them): the left segment belongs to waves 0-3,
//       the right to waves 4-7, and a wave owns blocks w, w + 4, ... (FP32
//       inputs are exact in FP64); from the same registers it also sums x over
//       its column blocks in FP64.
// The only barriers are those of the grouping, whose wait for all memory
// operations also lands the next tile's DMA issued one tile earlier.  Each
// wave carries its segment of the current cluster across tiles.  Slot mode
// (part != nullptr): a cluster that lies inside the workgroup's rows is
// written to its final place, the workgroup's first and last clusters that
// reach beyond them to partial slots 2 g and 2 g + 1 ([2][1 + E] each) that
// k_sub_stats_fix adds in a fixed order: no float atomics, so the sums do not
// depend on timing.  cstart / ctot are indexed by cluster - kbase.  Otherwise
// the segments are added to counts / moments with atomics.
// PAD: rows of d < D columns, copied four bytes per lane (a row need not be a
// multiple of 16 bytes); the columns from d on stay zero in LDS and their sums
// are dropped.  The generic kernel that this replaced kept 2 x 2 entries per
// lane and read two LDS operands per FMA: d = 100, N = 1e5, K = 32, sub-labels
// and statistics together 9.48 -> 0.17 ms; d = 127, N = 5e5, K = 16: 68.6 -> 0.52 ms.
template <int D, bool PAD>
__global__ __launch_bounds__(BIG_THREADS) void k_sub_stats_big(const float* __restrict__ x, int d, long long n_sorted,
                                                               int tpb, const int* __restrict__ perm,
                                                               const int* __restrict__ z,
                                                               const int* __restrict__ zrow,
                                                               const unsigned char* __restrict__ zsub,
                                                               long long* __restrict__ counts,
                                                               double* __restrict__ moments,
                                                               const int* __restrict__ cstart,
                                                               const int* __restrict__ ctot, int kbase,
                                                               double* __restrict__ part) {
  constexpr int R = big_rows_of(D);
  constexpr int NB = D / 16, NT = NB * (NB + 1) / 2, TPW = (NT + 3) / 4;
  const int dd = PAD ? d : D;  // columns of a row
  const int E = dd + dd * (dd + 1) / 2;
  constexpr int SB = D / 64;       // column blocks of sum x per wave
  constexpr int C4 = D / 4;        // 16-byte pieces per row
  constexpr int RPI = 64 / C4;     // rows per wave DMA instruction
  constexpr int NI = R / RPI / 8;  // DMA instructions per wave and tile
  static_assert(NI * RPI * 8 == R, "tile rows split evenly over the waves' DMA");
  // rows of two tiles, each followed by a zero row (read by lanes past a
  // segment).  Two arrays, and each tile's array fixed at compile time: the
  // compiler then knows that the rows a tile reads are not the ones its DMA
  // writes, and does not wait for the DMA before those reads.
  __shared__ float xa[(R + 1) * D], xb[(R + 1) * D];
  __shared__ int order[R], rk[R], buf[BIG_THREADS];
  __shared__ int lcount[2 * R], lstart[2 * R];
  __shared__ int rstart[R], ostart[R], rcl[R];
  __shared__ int nperm[2][R];  // point indices of the tiles whose rows are in flight
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int side = wave >> 2, wq = wave & 3;  // segment (0 left, 1 right), quarter
  int rd0, rd1;
  {
    const int i = lane & 15;
    if constexpr (D == 128) {
      const int s = ((i >> 2) ^ (i >> 3)) & 1;
      rd0 = 8 * i + 4 * s;
      rd1 = 8 * i + 4 * (1 - s);
    } else {
      rd0 = 4 * i;
      rd1 = rd0;
    }
  }
  const long long tiles = (n_sorted + R - 1) / R;
  const long long tb = (long long)blockIdx.x * tpb;
  const long long te = tb + tpb < tiles ? tb + tpb : tiles;
  const int nt = (int)(te - tb);
  const long long r_begin = tb * R;
  const long long r_end = te * R < n_sorted ? te * R : n_sorted;
  auto tile_rows = [&](int lt) __attribute__((always_inline)) -> int {
    const long long b = (tb + lt) * R;
    return (int)(n_sorted - b < R ? n_sorted - b : R);
  };
  f64x4 acc[TPW];
  double sx[SB];
  long long cnt_seg = 0;
  int cur_k = -1, k_first = -1;
  auto zero_acc = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < TPW; ++j) acc[j] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < SB; ++j) sx[j] = 0.0;
    cnt_seg = 0;
  };
  auto flush = [&]() __attribute__((always_inline)) {
    if (cur_k < 0) return;
    const int seg = 2 * cur_k + side;
    bool atomic = part == nullptr;
    double* M = moments + (size_t)seg * E;
    long long* C = counts + seg;
    double* Cd = nullptr;
    if (atomic) {
      if (cnt_seg == 0) return;
    } else {
      const long long cs = cstart[cur_k - kbase], ce = cs + ctot[cur_k - kbase];
      if (!(cs >= r_begin && ce <= r_end)) {
        double* P = part + ((size_t)(2 * blockIdx.x + (cur_k == k_first ? 0 : 1)) * 2 + side) * (E + 1);
        Cd = P;
        M = P + 1;
        C = nullptr;
      }
    }
#pragma unroll
    for (int j = 0; j < TPW; ++j) {
      // block (bI, bJ) of accumulator j: upper block wq + 4 j, row-major over I <= J
      int u = wq + 4 * j, bI = 0;
      if (u >= NT) continue;
      while (u >= NB - bI) {
        u -= NB - bI;
        ++bI;
      }
      const int bJ = bI + u;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        // accumulator element e of lane l is row l / 16 + 4 e, column l % 16
        // of block (I, J): the pair of columns col(I, row), col(J, column)
        const int ra = (lane >> 4) + 4 * e, rb = lane & 15;
        if (bI == bJ && ra > rb) continue;  // a diagonal block holds both orders
        const int c1 = big_col<D>(bI, ra), c2 = big_col<D>(bJ, rb);
        const int a = c1 < c2 ? c1 : c2, b = c1 < c2 ? c2 : c1;
        if (PAD && b >= dd) continue;
        double* dst = &M[dd + a * dd - (a * (a - 1)) / 2 + (b - a)];
        if (atomic)
          atomicAdd(dst, acc[j][e]);
        else
          *dst = acc[j][e];
      }
    }
#pragma unroll
    for (int j = 0; j < SB; ++j) {
      // the four row groups (lanes l, l + 16, l + 32, l + 48) combined
      double v = sx[j];
      v += __shfl_xor(v, 16);
      v += __shfl_xor(v, 32);
      if (lane < 16 && (!PAD || big_col<D>(wq + 4 * j, lane) < dd)) {
        double* dst = &M[big_col<D>(wq + 4 * j, lane)];
        if (atomic)
          atomicAdd(dst, v);
        else
          *dst = v;
      }
    }
    if (wq == 0 && lane == 0) {
      if (atomic)
        atomicAdd((unsigned long long*)C, (unsigned long long)cnt_seg);
      else if (C)
        *C = cnt_seg;
      else
        *Cd = (double)cnt_seg;
    }
  };
  // LDS DMA of tile lt's rows into dst, the point indices from nperm[lt % 2]
  auto issue_rows = [&](int lt, float* dst) __attribute__((always_inline)) {
    const int rows = tile_rows(lt);
    const int* np = nperm[lt & 1];
    if constexpr (PAD) {
      // 64 columns of a row per instruction; lanes past the columns copy nothing
#pragma unroll 8
      for (int i = 0; i < R * SB / 8; ++i) {
        const int r = (wave * (R * SB / 8) + i) / SB, c = (i % SB) * 64 + lane;
        if (c < dd)
          __builtin_amdgcn_global_load_lds((const void*)(x + (size_t)np[r < rows ? r : 0] * dd + c),
                                           (lds_void*)(dst + r * D + (i % SB) * 64), 4, 0, 0);
      }
      return;
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      // rows past the tile's end copy its first row (never read): no branches,
      // so the compiler's count of loads in flight stays exact
      const int r0 = (wave * NI + i) * RPI;
      const int r = r0 + lane / C4;
      __builtin_amdgcn_global_load_lds((const void*)(x + (size_t)np[r < rows ? r : 0] * D + 4 * (lane % C4)),
                                       (lds_void*)(dst + r0 * D), 16, 0, 0);
    }
  };
  zero_acc();
  // (k, zb: cluster and sub-label of row tid of the tile being grouped, loaded a
  // tile ahead and first used after the barrier that lands them)
  int k = -1;
  unsigned char zb = 0;
  if (nt > 0) {
    if (tid < tile_rows(0)) nperm[0][tid] = perm[r_begin + tid];
    for (int c = PAD ? tid : R * D + tid; c < (R + 1) * D; c += BIG_THREADS) {
      xa[c] = 0.0f;
      xb[c] = 0.0f;
    }
    __syncthreads();
    const int r = tid < tile_rows(0) ? tid : 0;
    const int mi = nperm[0][r];
    k = zrow ? zrow[r_begin + r] : z[mi];
    zb = zsub[mi];
    issue_rows(0, xa);
    if (nt > 1 && tid < tile_rows(1)) nperm[1][tid] = perm[r_begin + R + tid];
  }
  // one tile; its rows in xa (B = 0) or xb (B = 1), the next tile's DMA into the other
  auto tile_step = [&](auto bsel, auto wqc, int lt) __attribute__((always_inline)) {
    constexpr int B = decltype(bsel)::value;
    constexpr int WQ = decltype(wqc)::value;
    const float* tx = B ? xb : xa;
    float* nx = B ? xa : xb;
    const int rows = tile_rows(lt);
    const bool valid = tid < rows;
    // tile lt's rows and metadata have landed (the barrier waits for every memory
    // operation), the previous tile's LDS reads are done, nperm[(lt + 1) % 2] is visible
    __syncthreads();
    const int zs = zb ? 1 : 0;
    if (valid) rk[tid] = k;
    for (int q = tid; q < 2 * R; q += BIG_THREADS) lcount[q] = 0;
    __syncthreads();
    // ---- (2) group rows by segment: run of the cluster (rows are sorted by
    // z), then sub-label.  One scan gives the run of each row (high half) and
    // the right rows up to it (low half; both counts are <= R)
    const int zsv = valid ? zs : 0;
    const int flag = (valid && (tid == 0 || rk[tid] != rk[tid - 1])) ? 1 : 0;
    const int sc = block_inclusive_scan_big((flag << 16) | zsv, buf);
    const int run = (sc >> 16) - 1, ones_ex = (sc & 0xFFFF) - zsv;
    const int nruns = __builtin_amdgcn_readfirstlane(buf[BIG_THREADS - 1] >> 16);
    if (flag) {
      rstart[run] = tid;
      ostart[run] = ones_ex;
      rcl[run] = k;
    }
    const int lid = 2 * run + zsv;
    if (valid) atomicAdd(&lcount[lid], 1);  // integer counts: exact in any order
    __syncthreads();
    if (tid == 0) {
      int a = 0;
      for (int q = 0; q < 2 * nruns; ++q) {
        lstart[q] = a;
        a += lcount[q];
      }
    }
    __syncthreads();
    if (valid) {
      // rank among the run's rows of the same sub-label, in sorted order
      const int ones_run = ones_ex - ostart[run];
      const int rank = zsv ? ones_run : (tid - rstart[run]) - ones_run;
      order[lstart[lid] + rank] = tid;
    }
    __syncthreads();
    // ---- (1) the next tile: metadata into registers, the indices of the tile
    // after it, and its rows by DMA (the registers' first use is after the next
    // barrier, so nothing here waits for the DMA)
    int pn = -1;
    if (lt + 1 < nt) {
      const int r = tid < tile_rows(lt + 1) ? tid : 0;
      const int mi = nperm[(lt + 1) & 1][r];
      k = zrow ? zrow[(tb + lt + 1) * R + r] : z[mi];
      zb = zsub[mi];
      if (lt + 2 < nt) pn = perm[(tb + lt + 2) * R + (tid < tile_rows(lt + 2) ? tid : 0)];
      issue_rows(lt + 1, nx);
    }
    // ---- (3) every run, in order; this wave's side of it
    for (int j = 0; j < nruns; ++j) {
      const int kq = __builtin_amdgcn_readfirstlane(rcl[j]);
      if (kq != cur_k) {
        flush();
        zero_acc();
        if (cur_k < 0) k_first = kq;
        cur_k = kq;
      }
      const int q = 2 * j + side;
      const int cnt = __builtin_amdgcn_readfirstlane(lcount[q]);
      if (cnt == 0) continue;
      cnt_seg += cnt;
      const int st = __builtin_amdgcn_readfirstlane(lstart[q]);
      big_rows<D, WQ, R>(acc, sx, tx, order, st, cnt, lane, rd0, rd1);
    }
    // nperm[lt % 2] was last read before this tile's first barrier
    if (pn >= 0 && tid < R) nperm[lt & 1][tid] = pn;
  };
  // the tile loop once per quarter (a compile-time constant, so that its
  // blocks' operands are plain registers and the accumulators stay in place)
  auto run = [&](auto wqc) __attribute__((always_inline)) {
    for (int lt = 0; lt < nt; lt += 2) {
      tile_step(std::integral_constant<int, 0>{}, wqc, lt);
      if (lt + 1 < nt) tile_step(std::integral_constant<int, 1>{}, wqc, lt + 1);
    }
  };
  switch (wq) {
    case 0:
      run(std::integral_constant<int, 0>{});
      break;
    case 1:
      run(std::integral_constant<int, 1>{});
      break;
    case 2:
      run(std::integral_constant<int, 2>{});
      break;
    default:
      run(std::integral_constant<int, 3>{});
  }
  flush();
}

}  // namespace

hipError_t sorted_plan(long long n, int K, long long hist_cap, int* G, long long* per_block, int block_rows) {
  const SortedPlan p = plan_blocks(n, K, hist_cap, block_rows);
  *G = p.G;
  *per_block = p.per_block;
  return hipSuccess;
}

hipError_t launch_sort_by_z(const int* z, long long n, int K, int G, long long per_block, bool have_hist, int* hist,
                            int* tot, int* offs, int* perm, int* zsort, hipStream_t s, const int* mode) {
  if (n == 0) return hipSuccess;
  hipError_t e;
  if (G > SORT_BLOCKS) return hipErrorInvalidValue;
  if (!have_hist) {
    hipLaunchKernelGGL(k_hist_z, dim3(G), dim3(BLOCK), (size_t)K * sizeof(int), s, z, n, per_block, K, hist, mode);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_scan_hist, dim3(K), dim3(BLOCK), 0, s, hist, G, K, tot, offs, have_hist ? mode : nullptr);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // per_block is a multiple of BLOCK: each wave's quarter is whole 64-row chunks
  if (per_block % BLOCK != 0 || 4 * (size_t)K * sizeof(int) > 64 * 1024) return hipErrorInvalidValue;
  static bool attr_set = false;
  if (!attr_set) {  // the cursors of 4096 clusters take 64 KB beside the static scan buffer
    e = hipFuncSetAttribute((const void*)k_scatter_z, hipFuncAttributeMaxDynamicSharedMemorySize, 64 * 1024);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipLaunchKernelGGL(k_scatter_z, dim3(G), dim3(BLOCK), 4 * (size_t)K * sizeof(int), s, z, n, per_block, K, tot, offs,
                     perm, zsort, have_hist ? mode : nullptr);
  return hipGetLastError();
}

namespace {

// waves of k_sub_stats_w: the partial slots of 1024 ranges is what the other
// dimensions have always taken of the static scratch
int subw_waves(int d) { return d == 8 || d == 16 || d == 32 ? SUBW_WAVES : SUBW_WAVES / 2; }

// rows per wave of k_sub_stats_w (whole 64-row chunks, at most subw_waves(d) waves)
long long subw_rpw(int d, long long n) {
  long long rpw = (n + subw_waves(d) - 1) / subw_waves(d);
  return ((rpw + 63) / 64) * 64;
}

// columns of a row of k_sub_stats_big, zero-padded (d > 32)
int big_dim(int d) { return d <= 64 ? 64 : 128; }

// tiles per workgroup of k_sub_stats_big (at most 512 workgroups at d <= 64, 256 above)
int big_tpb(int d, long long n) {
  const int R = big_rows_of(big_dim(d));
  const long long tiles = (n + R - 1) / R;
  const long long gmax = d > 64 ? 256 : 512;
  const long long g = tiles < gmax ? tiles : gmax;
  return g > 0 ? (int)((tiles + g - 1) / g) : 1;
}

// The statistics kernels over rows perm[0, n) (point indices below npts).
// Slot mode (part != nullptr): cstart / ctot give the sorted start and size
// of clusters kbase ... kbase + ncl - 1 (indexed from 0), every one of their
// entries is written and nothing is added with atomics; otherwise the kernels
// add into counts / moments (which the caller has zeroed).
hipError_t sub_stats_kernels(int d, bool sample, const float* x, long long npts, long long n, const int* perm,
                             const int* z, const int* zrow, unsigned char* zsub, const float* packed, int K, int k_max,
                             uint32_t t, uint64_t seed, long long* counts, double* moments, const int* cstart,
                             const int* ctot, int kbase, int ncl, double* part, hipStream_t s,
                             const SubX3* x3 = nullptr) {
  hipError_t e;
  if (n == 0) return hipSuccess;
  const int E = d + d * (d + 1) / 2;
  const dim3 fix_grid((2 * (E + 1) + FIX_EN - 1) / FIX_EN, ncl);
  if (sample && d >= 32) {
    // the sub-labels in their own pass on the matrix cores, then the statistics.  With
    // BF16 tables (d = 64, 128) a bf16x3 pass draws most rows first and the FP32 kernel
    // only the list it leaves
    if (x3 && (d == 64 || d == 128)) {
      e = launch_sub_labels_x3(d, x, n, perm, z, zrow, zsub, packed, K, k_max, t, seed, *x3, s);
      if (e != hipSuccess) return e;
      e = launch_sub_labels_mx(d, x, n, x3->perm_c, nullptr, x3->zrow_c, zsub, packed, K, k_max, t, seed, s,
                               x3->offs + SUBX_GROUPS);
    } else {
      e = launch_sub_labels_mx(d, x, n, perm, z, zrow, zsub, packed, K, k_max, t, seed, s);
    }
    if (e != hipSuccess) return e;
    sample = false;
  }
  if (d > 32) {
    const int R = big_rows_of(big_dim(d));
    const long long tiles = (n + R - 1) / R;
    const int tpb = big_tpb(d, n);
    const unsigned grid = (unsigned)((tiles + tpb - 1) / tpb);
    const size_t lds = 0;  // all of its LDS is static (two tiles' rows, 129 KB)
#define DPMM_BIG(DD, PP)                                                                                          \
  hipLaunchKernelGGL((k_sub_stats_big<DD, PP>), dim3(grid), dim3(BIG_THREADS), lds, s, x, d, n, tpb, perm, z, zrow, \
                     zsub, counts, moments, cstart, ctot, kbase, part)
    if (d == 64)
      DPMM_BIG(64, false);
    else if (d == 128)
      DPMM_BIG(128, false);
    else if (d < 64)
      DPMM_BIG(64, true);
    else
      DPMM_BIG(128, true);
#undef DPMM_BIG
    if ((e = hipGetLastError()) != hipSuccess || !part) return e;
    hipLaunchKernelGGL(k_sub_stats_fix, fix_grid, dim3(FIX_PH * FIX_EN), 0, s, E, (long long)tpb * R, cstart,
                       ctot, part, counts, moments, kbase);
    return hipGetLastError();
  }
  {
    // four to eight waves per CU, each on a contiguous range of whole 64-row chunks
    const long long rpw = subw_rpw(d, n);
    const long long nw = (n + rpw - 1) / rpw;
    const unsigned grid = (unsigned)((nw + 3) / 4);
    const size_t lds = (size_t)4 * 64 * (d + 1) * sizeof(float);
#define DPMM_SUBW_CASE(DD)                                                                                      \
  case DD:                                                                                                      \
    if (sample)                                                                                                 \
      hipLaunchKernelGGL((k_sub_stats_w<DD, true>), dim3(grid), dim3(BLOCK), lds, s, x, npts, n, rpw, perm, z,  \
                         zrow, zsub, packed, K, k_max, t, seed, counts, moments, cstart, ctot, kbase, part);    \
    else                                                                                                        \
      hipLaunchKernelGGL((k_sub_stats_w<DD, false>), dim3(grid), dim3(BLOCK), lds, s, x, npts, n, rpw, perm, z, \
                         zrow, zsub, packed, K, k_max, t, seed, counts, moments, cstart, ctot, kbase, part);    \
    break;
    switch (d) {
      DPMM_SUBW_CASE(8)
      DPMM_SUBW_CASE(16)
      DPMM_SUBW_CASE(32)
      default:
        e = launch_sub_stats_w_any(d, sample, x, npts, n, rpw, perm, z, zrow, zsub, packed, K, k_max, t, seed, counts,
                                   moments, cstart, ctot, kbase, part, s);
        if (e != hipSuccess) return e;
    }
#undef DPMM_SUBW_CASE
    if ((e = hipGetLastError()) != hipSuccess || !part) return e;
    hipLaunchKernelGGL(k_sub_stats_fix, fix_grid, dim3(FIX_PH * FIX_EN), 0, s, E, rpw, cstart, ctot, part, counts,
                       moments, kbase);
    return hipGetLastError();
  }
}

}  // namespace

size_t sub_stats_part_doubles(int d, long long n) {
  const int E = d + d * (d + 1) / 2;
  long long ranges;
  if (n <= 0) return 0;
  if (d <= 32) {
    const long long rpw = subw_rpw(d, n);
    ranges = (n + rpw - 1) / rpw;
  } else {
    const int R = big_rows_of(big_dim(d));
    const long long tiles = (n + R - 1) / R;
    const int tpb = big_tpb(d, n);
    ranges = (tiles + tpb - 1) / tpb;
  }
  return (size_t)2 * ranges * 2 * (E + 1);
}

size_t sub_stats_part_doubles_max(int d) {
  const int E = d + d * (d + 1) / 2;
  const long long ranges = d <= 32 ? subw_waves(d) : (d > 64 ? 256 : 512);
  return (size_t)2 * ranges * 2 * (E + 1);
}

hipError_t launch_sub_stats(int d, bool sample, const float* x, long long n, const int* perm, const int* z,
                            const int* zrow, unsigned char* zsub, const float* packed, int K, int k_max, uint32_t t,
                            uint64_t seed, long long* counts, double* moments, const int* cstart, const int* ctot,
                            double* part, hipStream_t s, const SubX3* x3) {
  const int E = d + d * (d + 1) / 2;
  if (n > 0 && part)  // slot mode: every cluster's entries are written, no zeroing
    return sub_stats_kernels(d, sample, x, n, n, perm, z, zrow, zsub, packed, K, k_max, t, seed, counts, moments,
                             cstart, ctot, 0, K, part, s, x3);
  hipError_t e = launch_zero64(counts, (size_t)2 * K, s);
  if (e != hipSuccess) return e;
  e = launch_zero64(moments, (size_t)2 * K * E, s);
  if (e != hipSuccess) return e;
  return sub_stats_kernels(d, sample, x, n, n, perm, z, zrow, zsub, packed, K, k_max, t, seed, counts, moments,
                           nullptr, nullptr, 0, K, nullptr, s, x3);
}

bool partition_stats_supported(int d) { return d == 8 || d == 16 || d == 32 || d == 64 || d == 128; }

// The listed points idx[0, nsel) all belong to cluster k1; side[i] in {0, 1}
// plays the sub-label, so the sorted-order kernels leave the statistics of
// side h in segment 2 k1 + h of the arrays they are given.  Shifting the base
// pointers by slot - 2 k1 segments puts them in counts[slot + h] and
// moments[(slot + h) E] and touches nothing else.  cspan: device int[2] =
// {0, nsel} (the one cluster's sorted start and size); part: partial slots
// (sub_stats_part_doubles(d, nsel) doubles), summed in a fixed order.
hipError_t launch_partition_stats(int d, const float* x, long long npts, const int* idx, long long nsel,
                                  const int* z, int k1, int K, const unsigned char* side, int slot,
                                  long long* counts, double* moments, const int* cspan, double* part, hipStream_t s) {
  if (!partition_stats_supported(d) || k1 < 0 || k1 >= K || slot < 2 * k1 || !cspan || !part)
    return hipErrorInvalidValue;
  const int E = d + d * (d + 1) / 2;
  const long long shift = (long long)slot - 2 * k1;
  if (nsel == 0) {
    hipError_t e = launch_zero64(counts + slot, 2, s);
    if (e != hipSuccess) return e;
    return launch_zero64(moments + (size_t)slot * E, (size_t)2 * E, s);
  }
  return sub_stats_kernels(d, false, x, npts, nsel, idx, z, nullptr, const_cast<unsigned char*>(side), nullptr, K, 0,
                           0, 0, counts + shift, moments + shift * E, cspan, cspan + 1, k1, 1, part, s);
}

}  // namespace dpmm
