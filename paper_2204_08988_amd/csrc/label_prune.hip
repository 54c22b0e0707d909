// Gaussian cluster draw with clusters ruled out by their first whitened
// coordinates: Sec. 4.1 step (e), eq. sample_labels, for larger d, K, n.
//
// A cluster's squared norm q = fma(y_r, y_r, q) only grows with r, also in
// rounded arithmetic, so the score c - q / 2 of the first rows of W bounds the
// whole score from above.  A cluster whose bound lies below the leader's score by
// more than the Gumbel range cannot win, and its other rows need not be formed:
// for separated clusters 32 of d rows settle all but the point's own cluster.
//   k_pack_guess, k_guess   a guess of every point's cluster (the marginal density of
//                 the first 32 coordinates, in BF16 on the matrix cores) and, from the
//                 same products, an upper bound of the scores of all others;
//   the counting sort of the rows by guess (sorted.hip), so that the 64 points of a
//                 wave share theirs;
//   k_label_sorted  (FP32) per 256 sorted rows: their guessed clusters in full, which
//                 with the bound settles most points.  For the others every
//                 cluster's first 16 rows, then in full the clusters still in range
//                 for some point of the wave.  The draw of the points (score.hpp)
//                 takes the clusters in that order and gives the argmax of
//                 l_k + g_k with the smaller k on ties, as in increasing order;
//   k_sorted_x3   (BF16, label_mfma.hip) a lower bound of the guessed clusters' scores
//                 from bf16x3 products, which with the upper bound settles most points,
//                 and a list of the others for the main pass.
// FP32 scores have the bits of the kernel that forms them all (label_gauss_mx.hip), and
// what the bounds settle no score would change (interval.hpp), so the labels are the same
// whatever the data.  A BF16 draw, whose main pass over all points is within three times
// of this, first looks at 512 of the points (k_guess<true>) and takes that main pass
// where less than 3/4 of them would be settled.
//
// Label step (with sub-labels and statistics), all rows of every cluster -> so, us.
// FP32, means N(0, 9 I): d = 128, N = 1e6, K = 32 6080 -> 1233, N = 1e5, K = 64 1556 ->
// 393; d = 64, N = 5e5, K = 16 613 -> 308; d = 48, N = 1e5, K = 64 337 -> 144.  Where
// nearly every cluster stays in range of every point (means N(0, 0.01 I)) the extra
// passes cost 6% at d = 128, 21% at d = 64, 36% at d = 48.
// BF16: d = 128, N = 2e6, K = 100, means N(0, 9 I) 5414 -> 2630 (draw 3.3 -> 1.1 ms:
// guess 0.47, sort and probe 0.15, whole scores 0.27, open points 0.15), N(0, 2.25 I)
// 5854 and 5832, N(0, 0.09 I) 7234 and 7237; d = 64, N = 2e6, K = 200, N(0, 4 I) 3358
// -> 2240, N(0, 0.25 I) 4063 and 4051; N = 1e6, N(0, 0.25 I), where the look at the sample
// is 3 to 4%: K = 200 2190 and 2256, K = 64 984 and 1026.
#include "interval.hpp"
#include "kernels.hpp"
#include "score.hpp"
#include "score_mx.hpp"

namespace dpmm {

namespace {

using namespace score;

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

constexpr int GD = 32;  // coordinates of the guess
// one cluster's entry of the guess table: the BF16 fragments of W's first 32 rows
// ([2 k-steps][64 lanes][8]), the offsets -W (mu - c) in the accumulator layout
// ([2 lane halves][16]) and the constant
constexpr int GT_W = 2 * 64 * 8 * 2, GT_B = GD * 4, GT_BYTES = GT_W + GT_B + 16;
constexpr int GBLOCK = 256, GSTEP = 2 * GBLOCK;

// The table of every cluster, and after the K entries the common centre c (the
// mean of the first 64 cluster means: any centre will do, one near the data keeps
// the rounded rows small).
__global__ __launch_bounds__(128) void k_pack_guess(int K, int d, const float* __restrict__ packed,
                                                    unsigned char* __restrict__ tab, int* __restrict__ n_open) {
  __shared__ float cen[GD], part[4][GD];
  __shared__ float red[2];
  __shared__ double norm[2][2];
  if (blockIdx.x == 0 && threadIdx.x == 0) *n_open = 0;
  const int S = gauss_rec_stride(d), k = blockIdx.x, tid = threadIdx.x;
  {
    const int m = K < 64 ? K : 64, j = tid & (GD - 1), q0 = tid / GD;
    float s = 0.0f;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int c = q0 + 4 * q;
      s += c < m ? packed[(size_t)(c < m ? c : 0) * S + 4 + j] : 0.0f;
    }
    part[q0][j] = s;
    __syncthreads();
    if (tid < GD) {
      cen[tid] = (part[0][tid] + part[1][tid] + part[2][tid] + part[3][tid]) / (float)m;
      if (k == 0) reinterpret_cast<float*>(tab + (size_t)K * GT_BYTES)[tid] = cen[tid];
    }
  }
  __syncthreads();
  const float* rec = packed + (size_t)k * S;
  const float* w = rec + 4 + d;
  unsigned char* out = tab + (size_t)k * GT_BYTES;
  __bf16* fr = reinterpret_cast<__bf16*>(out);
  double wn = 0.0, mn = 0.0;
#pragma unroll
  for (int e0 = 0; e0 < 1024; e0 += 128) {
    const int e = e0 + tid, q = e & 7, lane = (e >> 3) & 63, ks = e >> 9;
    const int r = lane & 31, c = 16 * ks + 8 * (lane >> 5) + q;
    const float v = c <= r ? w[r * (r + 1) / 2 + c] : 0.0f;
    fr[e] = (__bf16)v;
    wn += (double)v * (double)v;
  }
  if (tid < GD) {
    float b = 0.0f;
    for (int c = 0; c <= tid; ++c) b = fmaf(w[tid * (tid + 1) / 2 + c], rec[4 + c] - cen[c], b);
    const int hh = (tid >> 2) & 1, j = ((tid >> 3) << 2) | (tid & 3);
    reinterpret_cast<float*>(out + GT_W)[hh * 16 + j] = -b;
    const double m = (double)rec[4 + tid] - (double)cen[tid];
    mn = m * m;
  }
  // log|W| of the rows left out, the norms of the first 32 rows
  float s = GD + tid < d ? logf(fabsf(w[(GD + tid) * (GD + tid + 1) / 2 + GD + tid])) : 0.0f;
  static_assert(PRUNE_MIN_D > GD, "rows are left out");
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    s += __shfl_xor(s, o);
    wn += __shfl_xor(wn, o);
    mn += __shfl_xor(mn, o);
  }
  if ((tid & 63) == 0) {
    red[tid >> 6] = s;
    norm[0][tid >> 6] = wn;
    norm[1][tid >> 6] = mn;
  }
  __syncthreads();
  if (tid == 0) {
    const double f = sqrt(norm[0][0] + norm[0][1]) * (1.0 + 1e-6);
    float4 c;
    c.x = rec[0] - (red[0] + red[1]);
    c.y = rec[0];
    c.z = (float)(((double)UC_GAMMA + (double)UC_GAMMA2) * f);
    c.w = (float)((double)UC_GAMMA2 * f * sqrt(norm[1][0] + norm[1][1]) * (1.0 + 1e-6));
    *reinterpret_cast<float4*>(out + GT_W + GT_B) = c;
  }
}

// Block b guesses the points [b per_block, (b + 1) per_block) and writes its
// histogram and, for each point, an upper bound of the FP32 scores of all clusters
// but the guessed one: c - max(0, s - E')^2 / 2 of the first 32 rows (interval.hpp),
// which a norm that only grows with the rows keeps; PR_REL covers the FP32
// evaluation of the bound.
//
// A wave takes 128 points (four 32-point tiles, rounded once), the tables come
// through LDS (all of them once, or groups in two buffers).  Bound by the vector
// ALUs and the matrix cores together (56 vector instructions per 64 points and
// cluster beside 4 matrix ones, 354 cycles; 64 points per wave, which double the LDS
// reads of the tables, and no bound took 392).  d = 64, N = 2e6, K = 200: 919 us (1004
// with groups of 16 clusters, two workgroups per CU instead of four): counters give the
// vector ALUs 80% and the matrix cores 45% of the cycles at the 1.86 GHz held; a tenth of
// the vector instructions less timed the same.
//
// mode (may be null): runs only where *mode is 1.  PROBE: one workgroup, the points
// 0, stride, ..., 511 stride, sets *mode to whether 3/4 of them would be settled by
// the bound, with d - 32 for the squared norm of a point's own remaining rows.
constexpr float PR_REL = 1e-6f;

template <bool PROBE>
__global__ __launch_bounds__(PROBE ? 2 * GBLOCK : GBLOCK, 2) void k_guess(const float* __restrict__ x, long long n, int d,
                                                     long long per_block, const unsigned char* __restrict__ tab, int K,
                                                     int cg, int* __restrict__ z, int* __restrict__ hist,
                                                     float* __restrict__ ub, int* mode, long long stride) {
  typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  // 32-point tiles of a wave (the single workgroup of the probe has twice the waves)
  constexpr int BLK = PROBE ? 2 * GBLOCK : GBLOCK, TILES = PROBE ? 2 : 4, OWN = TILES / 2;
  static_assert(BLK / 64 * 32 * TILES == GSTEP, "points per step");
  if (!PROBE && mode && *mode != 1) return;
  extern __shared__ __align__(16) unsigned char smem_g[];
  __shared__ int s_sure[BLK / 64];
  const bool single = cg >= K;
  unsigned char* buf0 = smem_g;
  unsigned char* buf1 = single ? smem_g : smem_g + cg * GT_BYTES;
  int* h = reinterpret_cast<int*>(smem_g + (single ? 1 : 2) * cg * GT_BYTES);
  if (!PROBE)
    for (int k = threadIdx.x; k < K; k += BLK) h[k] = 0;
  const int lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long long begin = (long long)blockIdx.x * per_block;
  const long long end = begin + per_block < n ? begin + per_block : n;
  auto fetch = [&](unsigned char* dst, int k0, int nk) {
    mx::stage<BLK>(reinterpret_cast<float*>(dst), reinterpret_cast<const float*>(tab + (size_t)k0 * GT_BYTES),
                      nk * (GT_BYTES / 4));
  };
  float cen[2][8];
  {
    const float* c = reinterpret_cast<const float*>(tab + (size_t)K * GT_BYTES);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int q = 0; q < 8; ++q) cen[ks][q] = c[16 * ks + 8 * half + q];
  }
  if (begin < end) fetch(buf0, 0, cg < K ? cg : K);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  int sure = 0;  // PROBE: the wave's points settled
  bool odd = false;
  for (long long chunk = begin; chunk < end; chunk += GSTEP) {
    const long long base = chunk + wave * 32 * TILES;
    bf16x8 b[TILES][2];  // [tile][k-step]
    float rx[TILES]; // the lane's half of ||x'||^2, then ||x'|| of its own two points
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
      const long long p = base + 32 * t + col;
      const bool ok = p < end;
      const float* xr = x + (ok ? (size_t)(PROBE ? p * stride : p) * d : 0) + 8 * half;
      rx[t] = 0.0f;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const f32x4u u = *reinterpret_cast<const f32x4u*>(xr + 16 * ks);
        const f32x4u v = *reinterpret_cast<const f32x4u*>(xr + 16 * ks + 4);
        const float f[8] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const float e = f[q] - cen[ks][q];
          rx[t] = fmaf(e, e, rx[t]);
          b[t][ks][q] = (__bf16)e;
        }
      }
    }
#pragma unroll
    for (int u = 0; u < OWN; ++u) rx[u] = __builtin_amdgcn_sqrtf(mx::half_sums(rx[2 * u], rx[2 * u + 1]));
    // points lane (and 64 + lane) of the wave: the best marginal, its cluster and its
    // bound, and the two largest bounds
    float best[OWN], mine[OWN], u1[OWN], u2[OWN], est[OWN];
    int arg[OWN];
#pragma unroll
    for (int u = 0; u < OWN; ++u) {
      best[u] = mine[u] = u1[u] = u2[u] = est[u] = -INFINITY;
      arg[u] = 0;
    }
    for (int g0 = 0; g0 < K; g0 += cg) {
      const int nk = K - g0 < cg ? K - g0 : cg;
      if (!single) {
        const bool wrap = g0 + cg >= K;
        const int gn = wrap ? 0 : g0 + cg;
        if (!wrap || chunk + GSTEP < end) fetch(odd ? buf0 : buf1, gn, K - gn < cg ? K - gn : cg);
      }
      typedef __attribute__((address_space(3))) const unsigned char lds_uchar;
      typedef __attribute__((address_space(3))) const bf16x8 lds_bf16x8;
      typedef __attribute__((address_space(3))) const f32x4 lds_f32x4;
      lds_uchar* e = (lds_uchar*)(odd ? buf1 : buf0);
      for (int c = 0; c < nk; ++c, e += GT_BYTES) {
        const bf16x8 a0 = ((lds_bf16x8*)e)[lane], a1 = ((lds_bf16x8*)e)[64 + lane];
        f32x16 off;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 u = ((lds_f32x4*)(e + GT_W))[4 * half + q];
#pragma unroll
          for (int j = 0; j < 4; ++j) off[4 * q + j] = u[j];
        }
        const f32x4 kc = *(lds_f32x4*)(e + GT_W + GT_B);
        float qs[TILES];
#pragma unroll
        for (int t = 0; t < TILES; ++t) {
          f32x16 acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, b[t][0], off, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, b[t][1], acc, 0, 0, 0);
          float q0 = 0.0f, q1 = 0.0f;
#pragma unroll
          for (int r = 0; r < 16; r += 2) {
            q0 = fmaf(acc[r], acc[r], q0);
            q1 = fmaf(acc[r + 1], acc[r + 1], q1);
          }
          qs[t] = q0 + q1;
        }
#pragma unroll
        for (int u = 0; u < OWN; ++u) {
          const float q = mx::half_sums(qs[2 * u], qs[2 * u + 1]);
          const float l = fmaf(-0.5f, q, kc.x), sq = __builtin_amdgcn_sqrtf(q);
          const float sm = fmaxf(sq - fmaf(UC_EPSS, sq, fmaf(kc.z, rx[u], kc.w)), 0.0f), h2 = 0.5f * sm * sm;
          const float up = fmaf(PR_REL, h2 + fabsf(kc.y), kc.y - h2);
          const bool better = l > best[u];
          arg[u] = better ? g0 + c : arg[u];
          mine[u] = better ? up : mine[u];
          if (PROBE) est[u] = better ? kc.y - 0.5f * (q + (float)(d - GD)) : est[u];
          best[u] = fmaxf(best[u], l);
          u2[u] = __builtin_amdgcn_fmed3f(u1[u], u2[u], up);
          u1[u] = fmaxf(u1[u], up);
        }
      }
      if (!single) {
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        odd = !odd;
      }
    }
#pragma unroll
    for (int u = 0; u < OWN; ++u) {
      const long long p = base + 64 * u + lane;
      const float other = mine[u] == u1[u] ? u2[u] : u1[u];
      if (PROBE) {
        sure += __popcll(__ballot(p < end && other < est[u] - RGAP));
      } else if (p < end) {
        z[p] = arg[u];
        ub[p] = other;
        atomicAdd(&h[arg[u]], 1);
      }
    }
  }
  if (PROBE && lane == 0) s_sure[wave] = sure;
  __syncthreads();
  if (PROBE) {
    if (threadIdx.x == 0) {
      int a = 0;
      for (int w = 0; w < BLK / 64; ++w) a += s_sure[w];
      *mode = 4 * a >= 3 * (int)(end - begin) ? 1 : 0;
    }
    return;
  }
  for (int k = threadIdx.x; k < K; k += BLK) hist[(size_t)blockIdx.x * K + k] = h[k];
}

constexpr int SBLOCK = 256;
constexpr int HEAD = 16;                                    // rows of W in a head
constexpr int HEAD_S = (4 + HEAD + HEAD * (HEAD + 1) / 2 + 3) & ~3;  // its record, as one of dimension 16
constexpr int HEAD_GROUP = 64;

// The draw of the rows sorted by guess, 256 per workgroup step.  LDS: one whole
// record, the heads of up to hg clusters (constant, first 16 means, first 16 rows
// of W), and per wave the clusters done and those still in range.  Bound by the
// FP32 matrix cores and the vector ALUs: per 64 points a whole evaluation (26 k
// cycles at d = 128: N = 2e6 0.42 ms, 2.5 TB/s of rows), and for a wave with a point that the guess's bound leaves open
// about 0.8 k cycles per cluster for the heads and the clusters in range in full.
template <int RB>
__global__ __launch_bounds__(SBLOCK, 2) void k_label_sorted(const float* __restrict__ x, long long n, int d,
                                                            const float* __restrict__ packed, int K, int hg,
                                                            const int* __restrict__ perm,
                                                            const int* __restrict__ guess, uint32_t t, uint64_t seed,
                                                            int* __restrict__ z, const float* __restrict__ ub) {
  extern __shared__ __align__(16) float smem_s[];
  __shared__ int s_k[SBLOCK];
  const int S = gauss_rec_stride(d), NW = (K + 31) >> 5;
  float* s_rec = smem_s;                                // a whole record
  float* s_head = smem_s + S + mx::REC_PAD;             // [hg] heads
  uint32_t* need = reinterpret_cast<uint32_t*>(s_head + hg * HEAD_S + mx::REC_PAD);  // [4][NW]
  uint32_t* done = need + 4 * NW;
  const int lane = threadIdx.x & 63, c16 = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t* my_need = need + wave * NW;
  uint32_t* my_done = done + wave * NW;
  mx::lds_cfloat* rec = (mx::lds_cfloat*)s_rec;
  for (long long chunk = (long long)blockIdx.x * SBLOCK; chunk < n; chunk += (long long)gridDim.x * SBLOCK) {
    const long long mine = chunk + threadIdx.x;
    const int i = mine < n ? perm[mine] : 0;
    const int k = mine < n ? guess[mine] : 0x7fffffff;
    float xv[4][4 * RB];
    const float* xr[4];
    bool ok[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = __shfl(i, 16 * q + c16);
      ok[q] = chunk + wave * 64 + 16 * q + c16 < n;
      xr[q] = x + (size_t)r * d;
    }
    mx::load_rows<RB>(xr, ok, d, xv);
    __syncthreads();  // the previous rows' tables are read
    s_k[threadIdx.x] = k;
    for (int w = threadIdx.x; w < 8 * NW; w += SBLOCK) need[w] = 0u;
    const float other = mine < n ? ub[i] : -INFINITY;  // what no other cluster exceeds
    bool open = mine < n;                              // a cluster beside those scored may win
    __syncthreads();
    StreamDraw dr;
    dr.init();
    auto whole = [&](int kk) __attribute__((always_inline)) {
      float q;
      const float cst = rec[0], fl = dr.floor();
      const bool full = mx::sq_norm<RB>(rec, d, xv, q, [&](float qp) {
        return __ballot(open && fmaf(-0.5f, qp, cst) > fl) != 0ull;
      });
      if (full) dr.push(fmaf(-0.5f, q, cst), kk, (uint32_t)i, t, seed);
    };
    auto fetch = [&](int kk) __attribute__((always_inline)) {
      __syncthreads();  // every wave is done with the previous record
      mx::stage<SBLOCK>(s_rec, packed + (size_t)kk * S, S);
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
    };
    // (1) the guessed clusters of the step's rows, then (3) those still in range:
    // one loop, so that the whole evaluation is instantiated once
    int w3 = -1;          // -1: phase (1); else the word of `need` being walked
    uint32_t bits = 0u;   // its clusters left (every wave's together)
    int cur = __builtin_amdgcn_readfirstlane(s_k[0]);
    for (;;) {
      bool eval;
      if (w3 < 0) {
        eval = __ballot(k == cur) != 0ull;
        if (eval && lane == 0) my_done[cur >> 5] |= 1u << (cur & 31);
      } else {
        eval = (__builtin_amdgcn_readfirstlane(my_need[cur >> 5] & ~my_done[cur >> 5]) >> (cur & 31)) & 1u;
      }
      fetch(cur);
      if (eval) whole(cur);
      if (w3 < 0) {
        // the next guessed cluster: the smallest above cur (every wave finds the same)
        int nx = 0x7fffffff;
#pragma unroll
        for (int q = 0; q < SBLOCK; q += 64) {
          const int v = s_k[q + lane];
          nx = v > cur && v < nx ? v : nx;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) nx = min(nx, __shfl_xor(nx, o));
        if (nx != 0x7fffffff) {
          cur = __builtin_amdgcn_readfirstlane(nx);
          continue;
        }
        open = open && !(other <= dr.floor());
        if (!__syncthreads_or(open)) break;
        // (2) the heads of all clusters
        float xh[4][4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int s = 0; s < 4; ++s) xh[q][s] = xv[q][s];
        const float fl = dr.floor();
        for (int g0 = 0; g0 < K; g0 += hg) {
          const int nk = K - g0 < hg ? K - g0 : hg;
          __syncthreads();  // the previous group is read
          for (int e0 = 0; e0 < nk * HEAD_S; e0 += SBLOCK) {
            const int e = e0 + threadIdx.x, q = e / HEAD_S, f = e - q * HEAD_S;
            if (q < nk && (f == 0 || (f >= 4 && f < 4 + HEAD + HEAD * (HEAD + 1) / 2)))
              __builtin_amdgcn_global_load_lds(
                  (const void*)(packed + (size_t)(g0 + q) * S + (f < 4 + HEAD ? f : f - HEAD + d)),
                  (mx::lds_void*)(s_head + (e & ~63)), 4, 0, 0);
          }
          __builtin_amdgcn_s_waitcnt(0);
          __syncthreads();
          mx::lds_cfloat* hp = (mx::lds_cfloat*)s_head;
          for (int c = 0; c < nk; ++c, hp += HEAD_S) {
            float q;
            mx::sq_norm<1>(hp, HEAD, xh, q, mx::Always());
            if (__ballot(open && fmaf(-0.5f, q, hp[0]) > fl) != 0ull && lane == 0)
              my_need[(g0 + c) >> 5] |= 1u << ((g0 + c) & 31);
          }
        }
        __syncthreads();  // every wave's clusters are marked
        w3 = 0;
        bits = 0u;
        cur = -1;
      }
      // the next cluster in range for some wave that has not had it
      while (bits == 0u && w3 <= NW - 1) {
        const int w = w3++;
        bits = __builtin_amdgcn_readfirstlane((need[w] & ~done[w]) | (need[NW + w] & ~done[NW + w]) |
                                              (need[2 * NW + w] & ~done[2 * NW + w]) |
                                              (need[3 * NW + w] & ~done[3 * NW + w]));
      }
      if (bits == 0u) break;
      const int bit = __builtin_ctz(bits);
      bits &= bits - 1;
      cur = 32 * (w3 - 1) + bit;
    }
    if (mine < n) z[i] = dr.finish((uint32_t)i, t, seed);
  }
}

}  // namespace

size_t guess_table_bytes(int d, int k_max) { return d >= PRUNE_MIN_D ? (size_t)k_max * GT_BYTES + GD * 4 : 0; }

// From the same comparison, us without and with, means N(0, 9 I): d = 40, N = 3e4,
// K = 16 86 and 89; d = 48, N = 3e4, K = 16 89 and 89, N = 8000, K = 32 133 and 119;
// N = 65536, K = 4: d = 64 97 and 111, d = 128 229 and 229.
// BF16, label step us without and with, means N(0, 9 I): d = 64, K = 20, N = 6e5 404 and
// 472, K = 64, N = 5e5 576 and 485; d = 128, N = 5e5, K = 8 705 and 735, K = 32 957 and 924.
// The look at the sample costs 0.4 us per cluster, which below 1e6 points shows where it
// decides against (d = 64, K = 64, N = 5e5, means N(0, I): 586 and 641).
bool label_prune_pays(int d, int K, long long n, bool bf16) {
  if (bf16) return n >= 1000000 && K >= (d >= 96 ? 32 : 64);
  return d >= PRUNE_MIN_D && K >= (d >= 96 ? 8 : 12) && n * K >= 250000;
}

hipError_t launch_guess(int d, const float* x, long long n, int G, long long per_block, const float* packed, int K,
                        const PruneBufs& b, bool probe, int* z, int* hist, hipStream_t s) {
  hipLaunchKernelGGL(k_pack_guess, dim3(K), dim3(128), 0, s, K, d, packed, b.tab, b.n_open);
  const int cg = K <= 16 ? K : 8;
  const size_t lds = (size_t)(K <= 16 ? 1 : 2) * cg * GT_BYTES + (size_t)K * sizeof(int);
  static bool attr_set = false;
  if (!attr_set) {
    for (const void* f : {(const void*)k_guess<true>, (const void*)k_guess<false>}) {
      const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024);
      if (e != hipSuccess) return e;
    }
    attr_set = true;
  }
  if (probe && n >= GSTEP)
    hipLaunchKernelGGL(k_guess<true>, dim3(1), dim3(2 * GBLOCK), lds, s, x, (long long)GSTEP, d, (long long)GSTEP, b.tab, K,
                       cg, z, hist, b.ub, b.mode, n / GSTEP);
  hipLaunchKernelGGL(k_guess<false>, dim3(G), dim3(GBLOCK), lds, s, x, n, d, per_block, b.tab, K, cg, z, hist, b.ub,
                     probe ? b.mode : nullptr, 1ll);
  return hipGetLastError();
}

hipError_t launch_label_sorted(int d, const float* x, long long n, const float* packed, int K, const int* perm,
                               const int* guess, uint32_t t, uint64_t seed, const float* ub, int* z, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const int hg = K < HEAD_GROUP ? K : HEAD_GROUP;
  const size_t lds = (size_t)(gauss_rec_stride(d) + hg * HEAD_S + 2 * mx::REC_PAD) * sizeof(float) +
                     (size_t)8 * ((K + 31) / 32) * sizeof(uint32_t);
  static bool attr_set = false;
  if (!attr_set) {
    const void* fns[6] = {(const void*)k_label_sorted<3>, (const void*)k_label_sorted<4>,
                          (const void*)k_label_sorted<5>, (const void*)k_label_sorted<6>,
                          (const void*)k_label_sorted<7>, (const void*)k_label_sorted<8>};
    for (const void* f : fns) {
      const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024);
      if (e != hipSuccess) return e;
    }
    attr_set = true;
  }
  const unsigned G = (unsigned)((n + SBLOCK - 1) / SBLOCK < 65536 ? (n + SBLOCK - 1) / SBLOCK : 65536);
#define DPMM_SORTED(RB)                                                                                              \
  hipLaunchKernelGGL(k_label_sorted<RB>, dim3(G), dim3(SBLOCK), lds, s, x, n, d, packed, K, hg, perm, guess, t, seed, \
                     z, ub)
  switch (mx::row_blocks(d)) {
    case 3: DPMM_SORTED(3); break;
    case 4: DPMM_SORTED(4); break;
    case 5: DPMM_SORTED(5); break;
    case 6: DPMM_SORTED(6); break;
    case 7: DPMM_SORTED(7); break;
    case 8: DPMM_SORTED(8); break;
    default: return hipErrorInvalidValue;
  }
#undef DPMM_SORTED
  return hipGetLastError();
}

}  // namespace dpmm
