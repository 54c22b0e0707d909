// Label step of dense counts in float32: Sec. 4.1 steps (e) and (f) with
// multinomial components (Sec. 2.1; Poisson ones score alike).
//
// Score of a component: l = log w + sum_v x_v log theta_v (the multinomial
// coefficient is the same for every component and is left out).  Two kernels:
// k_label_mult_mfma on the FP32 matrix cores while log theta of all clusters fits
// in LDS, and for more of them k_label_mult, one lane per point: the count row is
// converted to float32 once (counts below 2^24 are exact) and held in registers, the
// uniform cluster loop reads log theta with scalar loads; label and sub-label draws as in
// the Gaussian kernel: top-2 screen, lazy Gumbel-max, logistic skipped outside its
// range.
#include "kernels.hpp"
#include "score_mx.hpp"

namespace dpmm {

namespace {

constexpr int BLOCK = 256;
constexpr float RGAP = GUMBEL_MAX_F - GUMBEL_MIN_F;
constexpr size_t MULT_MFMA_LDS_MAX = 96 * 1024;  // log theta staged for every cluster

// orders the wave's own LDS accesses (no workgroup barrier)
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int VT>
__device__ __forceinline__ float score_mult(const float* __restrict__ p, const float (&x)[VT]) {
  float a0 = p[0], a1 = 0.0f;
#pragma unroll
  for (int v = 0; v < VT; v += 2) {
    a0 = fmaf(x[v], p[4 + v], a0);
    if (v + 1 < VT) a1 = fmaf(x[v + 1], p[5 + v], a1);
  }
  return a0 + a1;
}

template <int VT>
__global__ __launch_bounds__(BLOCK) void k_label_mult(const int* __restrict__ x, long long n, int V,
                                                      const float* __restrict__ packed, int K, int k_max,
                                                      uint32_t t, uint64_t seed, int* __restrict__ z,
                                                      unsigned char* __restrict__ zsub) {
  const int S = mult_rec_stride(V);
  const long long stride_pts = (long long)gridDim.x * BLOCK;
  for (long long i = (long long)blockIdx.x * BLOCK + threadIdx.x; i < n; i += stride_pts) {
    // unconditional loads (clamped word index, zeroed afterwards): all in flight together
    float xv[VT];
#pragma unroll
    for (int v = 0; v < VT; ++v) {
      const int c = x[i * V + (v < V ? v : V - 1)];
      xv[v] = v < V ? (float)c : 0.0f;
    }
    float m1 = -INFINITY, m2 = -INFINITY;
    int arg = 0;
    for (int k = 0; k < K; ++k) {
      const float l = score_mult<VT>(packed + (size_t)k * S, xv);
      if (l > m1) {
        m2 = m1;
        m1 = l;
        arg = k;
      } else if (l > m2) {
        m2 = l;
      }
    }
    int zi = arg;
    if (m2 > m1 - RGAP) {
      int cached = arg >> 2;
      u32x4 blk = rng_block(seed, t, (uint32_t)i, TAG_GUMBEL, (uint32_t)cached);
      float best = m1 + gumbel_f(word_of(blk, arg & 3));
      for (int k = 0; k < K; ++k) {
        if (k == arg) continue;
        const float l = score_mult<VT>(packed + (size_t)k * S, xv);
        if (l + GUMBEL_MAX_F > best) {
          const int b = k >> 2;
          if (b != cached) {
            blk = rng_block(seed, t, (uint32_t)i, TAG_GUMBEL, (uint32_t)b);
            cached = b;
          }
          const float s = l + gumbel_f(word_of(blk, k & 3));
          if (s > best || (s == best && k < zi)) {
            best = s;
            zi = k;
          }
        }
      }
    }
    const float* ps = packed + (size_t)(k_max + 2 * zi) * S;
    const float delta = score_mult<VT>(ps, xv) - score_mult<VT>(ps + S, xv);
    unsigned char zs;
    zs = sub_label_draw(delta, seed, t, (uint32_t)i, K);
    z[i] = zi;
    zsub[i] = zs;
  }
}

// The same draw with the scores on the FP32 matrix cores: v_mfma_f32_16x16x4_f32
// adds its products one after the other in increasing word order (score_mx.hpp),
// so a score is the chain l = fma(x_v, log theta_v, l) from l = log w.  A wave
// takes 64 points (four 16-point tiles, rows in registers as in score_mx.hpp)
// against groups of 64 clusters: A = log theta (staged in LDS for all K clusters
// once per workgroup, rows of 4 x odd floats: the sixteen rows x four words of a
// read fall on 64 banks), B = the counts.  Lane 16 g + c of a tile ends with the
// clusters 4 g .. 4 g + 3 of every 16 for point c.
//
// Clusters within the Gumbel range of the running maximum are listed per wave in
// LDS by fours (point, the clusters of one random block and their scores); with a
// single group only those of points that have several.  A lane draws the Gumbels of
// one entry, whatever point it belongs to, and each point's winner (largest l_k +
// g_k, smaller k on ties) is a 64-bit LDS maximum: a wave with a few doubtful points
// pays for their clusters, not for every cluster of 64 points, and one whose clusters
// are nearly all in range for one random block per four of them.  The sub-label needs
// the point's whole row on one lane: a 4 x 4 lane transpose of the registers.  The two
// sub-cluster records come from LDS while they fit beside the clusters'.
//
// Bound by the FP32 matrix cores, and HBM behind them.  N = 1e6, V = 100, K = 50:
// 646 us (32-row tiles, rows read with a stride, the whole wave scored twice for
// one doubtful point, sub-cluster records gathered from memory) -> 186 us; its 400
// matrix instructions per 64 points take 95.  With nearly every cluster in range (counts
// of one law) V = 7, K = 200, N = 3e5: 233 us that way, 365 with the candidates listed
// one by one and a random block for each, 182 so; V = 64, K = 300, N = 5e4: 130, 210, 94.
constexpr int MM_BLOCK = 512;  // threads at most
constexpr int MM_LIST = 256;  // fours of candidates listed per wave: those of one tile and group always fit
constexpr size_t MM_LDS_MAX = 150 * 1024;
// up to here workgroups of half as many threads, so that no more than one per CU
// still leaves fewer CUs idle: V = 100, K = 50, us with 256 and 512 threads: n = 2e4 30 and
// 39, 5e4 31 and 40, 1e5 58 and 43; V = 32, K = 600: n = 5e4 150 and 192, 1e5 285 and 200
constexpr long long MM_SMALL_N = 65536;

__host__ __device__ constexpr int mm_ldv(int V) { return 4 * (((V + 3) / 4) | 1); }

// A float in an order-preserving 32-bit key.
__device__ __forceinline__ uint32_t order_key(float v) {
  const uint32_t b = __float_as_uint(v);
  return b & 0x80000000u ? ~b : b | 0x80000000u;
}

template <int RB, bool SUB>
__global__ __launch_bounds__(MM_BLOCK, 2) void k_label_mult_mfma(const int* __restrict__ x, long long n, int V,
                                                                 const float* __restrict__ packed, int K, int k_max,
                                                                 uint32_t t, uint64_t seed,
                                                                 int* __restrict__ z, unsigned char* __restrict__ zsub) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  const int nt = blockDim.x, nw = nt / 64;
  const int S = mult_rec_stride(V), LDV = mm_ldv(V), Q = LDV / 4;
  extern __shared__ __align__(16) float th[];  // [K][LDV] clusters, then (SUB) [2K][LDV] sub-clusters
  float* cw = th + (size_t)(SUB ? 3 : 1) * K * LDV;  // [K rounded up to 64] log w (-inf past K), [2K] sub-clusters'
  const int KP = (K + 63) & ~63;
  f32x4* lists = reinterpret_cast<f32x4*>(cw + KP);  // [waves][MM_LIST] scores of clusters k .. k + 3
  unsigned long long* best_all = reinterpret_cast<unsigned long long*>(lists + nw * MM_LIST);  // [waves][64]
  float* csub = reinterpret_cast<float*>(best_all + nw * 64);
  unsigned short* listk = reinterpret_cast<unsigned short*>(csub + 2 * K);  // [waves][MM_LIST] point << 10 | k
  {
    const int rows = SUB ? 3 * K : K;
    for (int e = threadIdx.x; e < rows * Q; e += nt) {
      const int r = e / Q, q = e - r * Q;
      const float* src = packed + (size_t)(r < K ? r : k_max + (r - K)) * S + 4;
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (4 * q < V) v = *reinterpret_cast<const float4*>(src + 4 * q);
      v.x = 4 * q < V ? v.x : 0.0f;
      v.y = 4 * q + 1 < V ? v.y : 0.0f;
      v.z = 4 * q + 2 < V ? v.z : 0.0f;
      v.w = 4 * q + 3 < V ? v.w : 0.0f;
      *reinterpret_cast<float4*>(th + (size_t)r * LDV + 4 * q) = v;
    }
    for (int k = threadIdx.x; k < KP; k += nt) cw[k] = k < K ? packed[(size_t)k * S] : -INFINITY;
    for (int k = threadIdx.x; k < 2 * K; k += nt) csub[k] = packed[(size_t)(k_max + k) * S];
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  unsigned long long* best = best_all + wave * 64;
  f32x4* ll = lists + wave * MM_LIST;
  unsigned short* lk = listk + wave * MM_LIST;
  const int ext = V - 16 * (RB - 1);  // words of the last 16
  // Gumbels of the listed candidates above their point's floor; the winners into best
  auto draw_list = [&](int cnt, const float (&fl)[4], long long base) __attribute__((always_inline)) {
    wave_sync();
    for (int e0 = 0; e0 < cnt; e0 += 64) {
      const int e = e0 + lane;
      const f32x4 l = ll[e < cnt ? e : 0];
      const int pk = lk[e < cnt ? e : 0], p = pk >> 10, k = pk & 1023;
      // the floor of point p: lane p % 16 holds it for tile p / 16
      const float f0 = __shfl(fl[0], p & 15), f1 = __shfl(fl[1], p & 15), f2 = __shfl(fl[2], p & 15),
                  f3 = __shfl(fl[3], p & 15);
      const float f = p < 32 ? (p < 16 ? f0 : f1) : (p < 48 ? f2 : f3);
      if (e < cnt && (l[0] > f || l[1] > f || l[2] > f || l[3] > f)) {
        const u32x4 blk = rng_block(seed, t, (uint32_t)(base + p), TAG_GUMBEL, (uint32_t)(k >> 2));
        float sv = -INFINITY;
        int w = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (l[u] > f) {
            const float v = l[u] + gumbel_f(word_of(blk, u));
            w = v > sv ? u : w;  // the smaller k on ties
            sv = fmaxf(sv, v);
          }
        atomicMax(&best[p], (unsigned long long)order_key(sv) << 32 | (uint32_t)(0x7fffffff - (k + w)));
      }
    }
    wave_sync();
  };
  for (long long chunk = (long long)blockIdx.x * nt; chunk < n; chunk += (long long)gridDim.x * nt) {
    const long long base = chunk + wave * 64;
    if (base >= n) continue;  // (no workgroup barrier in the loop)
    float xv[4][4 * RB];
    {
      const float* xr[4];
      bool ok[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const long long p = base + 16 * q + c;
        ok[q] = p < n;
        xr[q] = reinterpret_cast<const float*>(x) + (ok[q] ? (size_t)p * V : 0);
      }
      mx::load_rows<RB>(xr, ok, V, xv);
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int s = 0; s < 4 * RB; ++s) xv[q][s] = (float)__float_as_int(xv[q][s]);
    }
    best[lane] = 0ull;  // below the key of every score
    float m1[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};  // maxima of point c of each tile
    float fl[4];
    int arg[4] = {0, 0, 0, 0};  // the leader, the smallest k on ties
    bool many[4] = {false, false, false, false};
    int cnt = 0;
    for (int k0 = 0; k0 < K; k0 += 64) {
      f32x4 a[4][4];  // [row block][tile]
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) {
        const f32x4 c0 = *reinterpret_cast<const f32x4*>(cw + k0 + 16 * rb + 4 * g);
#pragma unroll
        for (int q = 0; q < 4; ++q) a[rb][q] = c0;
      }
      // row block by row block; W is read PF steps ahead of its use
      constexpr int PF = 4;
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) {
        if (rb > 0 && k0 + 16 * rb >= K) continue;
        const int r = k0 + 16 * rb + c;
        mx::lds_cfloat* wr = (mx::lds_cfloat*)th + (r < K ? r : K - 1) * LDV + g;
        float w[4 * RB];
#pragma unroll
        for (int s = 0; s < PF && s < 4 * RB; ++s) w[s] = wr[4 * s];
#pragma unroll
        for (int s = 0; s < 4 * RB; ++s) {
          // (rows are padded to LDV >= V; reads past them stay inside LDS and are not used)
          if (s + PF < 4 * RB) w[s + PF] = wr[4 * (s + PF)];
          __builtin_amdgcn_sched_barrier(0);
          if (s <= 4 * (RB - 1) || 4 * (s - 4 * (RB - 1)) < ext) {  // steps past the last word: skipped (uniform)
#pragma unroll
            for (int q = 0; q < 4; ++q)
              a[rb][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[s], xv[q][s], a[rb][q], 0, 0, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        // the point's maximum over this lane's 16 clusters, then over the four lane groups
        float b = -INFINITY;
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) b = fmaxf(b, fmaxf(fmaxf(a[rb][q][0], a[rb][q][1]), fmaxf(a[rb][q][2], a[rb][q][3])));
        b = fmaxf(b, __shfl_xor(b, 16));
        b = fmaxf(b, __shfl_xor(b, 32));
        const bool higher = b > m1[q];
        m1[q] = fmaxf(m1[q], b);
        fl[q] = m1[q] - RGAP;
        int in = 0, kk = 0x7fffffff;
#pragma unroll
        for (int rb = 3; rb >= 0; --rb)
#pragma unroll
          for (int u = 3; u >= 0; --u) {
            in += a[rb][q][u] > fl[q] ? 1 : 0;
            kk = a[rb][q][u] == m1[q] ? k0 + 16 * rb + 4 * g + u : kk;
          }
        kk = min(kk, __shfl_xor(kk, 16));
        kk = min(kk, __shfl_xor(kk, 32));
        arg[q] = higher ? kk : arg[q];
        if (K <= 64) {  // the only group: clusters in range of the point
          int tot = in + __shfl_xor(in, 16);
          tot += __shfl_xor(tot, 32);
          many[q] = tot > 1;
        } else {
          many[q] = true;
        }
        const bool list_it = many[q] && in > 0 && base + 16 * q + c < n;
        if (__ballot(list_it)) {
          bool up[4];
          int add = 0;
#pragma unroll
          for (int rb = 0; rb < 4; ++rb) {
            const f32x4 v = a[rb][q];
            up[rb] = list_it && (v[0] > fl[q] || v[1] > fl[q] || v[2] > fl[q] || v[3] > fl[q]);
            add += __popcll(__ballot(up[rb]));
          }
          if (cnt + add > MM_LIST) {
            draw_list(cnt, fl, base);
            cnt = 0;
          }
#pragma unroll
          for (int rb = 0; rb < 4; ++rb) {
            const unsigned long long m = __ballot(up[rb]);
            if (up[rb]) {
              const int o = cnt + __popcll(m & ((1ull << lane) - 1ull));
              ll[o] = a[rb][q];
              lk[o] = (unsigned short)((16 * q + c) << 10 | (k0 + 16 * rb + 4 * g));
            }
            cnt += __popcll(m);
          }
        }
      }
    }
    if (cnt) draw_list(cnt, fl, base);
    // the lane's own point: tile g, point c
    int zi = g == 0 ? arg[0] : (g == 1 ? arg[1] : (g == 2 ? arg[2] : arg[3]));
    const bool drew = g == 0 ? many[0] : (g == 1 ? many[1] : (g == 2 ? many[2] : many[3]));
    if (drew) {
      const unsigned long long bk = best[lane];
      if (bk) zi = 0x7fffffff - (int)(uint32_t)bk;  // (0: scores so large that the range vanishes in them)
    }
    wave_sync();  // best is reset by the next rows
    // its sub-label: word v on even and odd chains, as score_mult
#pragma unroll
    for (int s = 0; s < 4 * RB; ++s) mx::transpose4(xv[0][s], xv[1][s], xv[2][s], xv[3][s]);  // word 4 s + q in xv[q][s]
    const long long i = base + lane;
    float sc[2];
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      float a0 = csub[2 * zi + hh], a1 = 0.0f;
      if constexpr (SUB) {
        // (words past V: zeros on both sides, which leave the chains as they are)
        typedef __attribute__((address_space(3))) const f32x4 lds_f32x4;
        lds_f32x4* ps = (lds_f32x4*)(th + (size_t)(K + 2 * zi + hh) * LDV);
#pragma unroll
        for (int s = 0; s < 4 * RB; ++s) {
          if (s > 4 * (RB - 1) && 4 * (s - 4 * (RB - 1)) >= ext) continue;
          const f32x4 w = ps[s];
          a0 = fmaf(xv[0][s], w[0], a0);
          a1 = fmaf(xv[1][s], w[1], a1);
          a0 = fmaf(xv[2][s], w[2], a0);
          a1 = fmaf(xv[3][s], w[3], a1);
        }
      } else {
        const float* ps = packed + (size_t)(k_max + 2 * zi + hh) * S + 4;
#pragma unroll
        for (int s = 0; s < 4 * RB; ++s) {
          if (s > 4 * (RB - 1) && 4 * (s - 4 * (RB - 1)) >= ext) continue;
          const float4 w = *reinterpret_cast<const float4*>(ps + 4 * s);
          const bool tail = s >= 4 * (RB - 1);  // words past V are not the record's
          a0 = fmaf(xv[0][s], w.x, a0);
          a1 = !tail || 4 * s + 1 < V ? fmaf(xv[1][s], w.y, a1) : a1;
          a0 = !tail || 4 * s + 2 < V ? fmaf(xv[2][s], w.z, a0) : a0;
          a1 = !tail || 4 * s + 3 < V ? fmaf(xv[3][s], w.w, a1) : a1;
        }
      }
      sc[hh] = a0 + a1;
    }
    if (i < n) {
      z[i] = zi;
      zsub[i] = (unsigned char)sub_label_draw(sc[0] - sc[1], seed, t, (uint32_t)i, K);
    }
  }
}

size_t label_mult_mfma_lds(int V, int K, bool sub, int nt) {
  return ((size_t)(sub ? 3 : 1) * K * mm_ldv(V) + ((K + 63) & ~63) + 2 * (size_t)K) * sizeof(float) +
         (size_t)(nt / 64) * (64 * sizeof(unsigned long long) + MM_LIST * (4 * sizeof(float) + sizeof(unsigned short)));
}

// The matrix-core draw takes the calls whose log theta, in rows of 32, 64 or 128
// words and blocks of 32 clusters, fits 96 KB (K <= 704, 352, 160).  The two
// draws round their scores differently, so the line stays where it has been: a
// call keeps its labels.
bool mult_on_matrix_cores(int V, int K) {
  const int VH = V <= 32 ? 16 : (V <= 64 ? 32 : 64);
  const size_t kb = (size_t)(K + 31) / 32;
  return V <= 128 && (kb * 32 * (2 * VH + 1) + kb * 32) * sizeof(float) <= MULT_MFMA_LDS_MAX;
}

__global__ __launch_bounds__(BLOCK) void k_loglik_mult(const int* __restrict__ x, long long n, int V,
                                                       const float* __restrict__ packed, int K, int k_max,
                                                       float* __restrict__ out) {
  const int S = mult_rec_stride(V);
  const long long stride_pts = (long long)gridDim.x * BLOCK;
  for (long long i = (long long)blockIdx.x * BLOCK + threadIdx.x; i < n; i += stride_pts) {
    const int* xi = x + i * V;
    float* o = out + i * 3 * K;
    for (int j = 0; j < 3 * K; ++j) {
      const int slot = j < K ? j : k_max + (j - K);
      const float* p = packed + (size_t)slot * S;
      float a = p[0];
      for (int v = 0; v < V; ++v) a = fmaf((float)xi[v], p[4 + v], a);
      o[j] = a;
    }
  }
}

int grid_for(long long n) {
  long long g = (n + BLOCK - 1) / BLOCK;
  if (g > 8192) g = 8192;
  if (g < 1) g = 1;
  return (int)g;
}

}  // namespace

hipError_t launch_label_mult(int V, const int* x, long long n, const float* packed, int K, int k_max,
                             uint32_t t, uint64_t seed, int* z, unsigned char* zsub, hipStream_t s) {
  if (n == 0) return hipSuccess;
  if (mult_on_matrix_cores(V, K)) {
    const int nt = n <= MM_SMALL_N ? MM_BLOCK / 2 : MM_BLOCK;
    const bool sub = label_mult_mfma_lds(V, K, true, nt) <= MM_LDS_MAX;
    const size_t lds = label_mult_mfma_lds(V, K, sub, nt);
    static bool attr_set = false;
    if (!attr_set) {
      const void* fns[16] = {
          (const void*)k_label_mult_mfma<1, true>,  (const void*)k_label_mult_mfma<2, true>,
          (const void*)k_label_mult_mfma<3, true>,  (const void*)k_label_mult_mfma<4, true>,
          (const void*)k_label_mult_mfma<5, true>,  (const void*)k_label_mult_mfma<6, true>,
          (const void*)k_label_mult_mfma<7, true>,  (const void*)k_label_mult_mfma<8, true>,
          (const void*)k_label_mult_mfma<1, false>, (const void*)k_label_mult_mfma<2, false>,
          (const void*)k_label_mult_mfma<3, false>, (const void*)k_label_mult_mfma<4, false>,
          (const void*)k_label_mult_mfma<5, false>, (const void*)k_label_mult_mfma<6, false>,
          (const void*)k_label_mult_mfma<7, false>, (const void*)k_label_mult_mfma<8, false>};
      for (const void* f : fns) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
      }
      attr_set = true;
    }
    // one workgroup per CU, which stages the tables once
    long long g = (n + nt - 1) / nt;
    if (g > 256) g = 256;
#define DPMM_MM_CASE(RB)                                                                                              \
  case RB:                                                                                                            \
    if (sub)                                                                                                          \
      hipLaunchKernelGGL((k_label_mult_mfma<RB, true>), dim3(g), dim3(nt), lds, s, x, n, V, packed, K, k_max, t, \
                         seed, z, zsub);                                                                              \
    else                                                                                                              \
      hipLaunchKernelGGL((k_label_mult_mfma<RB, false>), dim3(g), dim3(nt), lds, s, x, n, V, packed, K, k_max, t, \
                         seed, z, zsub);                                                                              \
    break;
    switch (mx::row_blocks(V)) {
      DPMM_MM_CASE(1)
      DPMM_MM_CASE(2)
      DPMM_MM_CASE(3)
      DPMM_MM_CASE(4)
      DPMM_MM_CASE(5)
      DPMM_MM_CASE(6)
      DPMM_MM_CASE(7)
      DPMM_MM_CASE(8)
      default:
        return hipErrorInvalidValue;
    }
#undef DPMM_MM_CASE
    return hipGetLastError();
  }
  const int g = grid_for(n);
  if (V <= 32) {
    hipLaunchKernelGGL(k_label_mult<32>, dim3(g), dim3(BLOCK), 0, s, x, n, V, packed, K, k_max, t, seed, z, zsub);
  } else if (V <= 64) {
    hipLaunchKernelGGL(k_label_mult<64>, dim3(g), dim3(BLOCK), 0, s, x, n, V, packed, K, k_max, t, seed, z, zsub);
  } else if (V <= 128) {
    hipLaunchKernelGGL(k_label_mult<128>, dim3(g), dim3(BLOCK), 0, s, x, n, V, packed, K, k_max, t, seed, z,
                       zsub);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_loglik_mult(int V, const int* x, long long n, const float* packed, int K, int k_max,
                              float* out, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_loglik_mult, dim3(grid_for(n)), dim3(BLOCK), 0, s, x, n, V, packed, K, k_max, out);
  return hipGetLastError();
}

}  // namespace dpmm
