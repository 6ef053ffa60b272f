/*
 * abea_meth.hip -- gfx950 kernels of methylation scoring, the step after the
 * alignment: the events aligned to the reference's k-mers go through HMM
 * profiling to decide whether a base is methylated (the thesis, Ch. 5
 * §5.2.2 "Methylation calling"; it gives no algorithm for the profile).
 *
 * The profile:
 *   - a site is a CpG whose C starts k-mer i of a read (the first two bases
 *     of k-mer i are C, G); its window is the k-mers holding that C,
 *     j0 = max(0, i-k+1) .. i;
 *   - the window's events run from the first event the alignment paired with
 *     k-mer j0 to the last it paired with k-mer i;
 *   - under each of two models (the context's pore model and the methylated
 *     one) the best-path score of those events through the window's k-mers,
 *     with the alignment's own cell score (Alg. 5.2 moves with the read's
 *     transition constants, Alg. 5.3 emission, the model scaled per read): a
 *     virtual origin before the first cell scores 0, cells outside the window
 *     are -inf, and the score is the last cell's;
 *   - LLR = score(methylated) - score(unmethylated), float32.
 *
 * Kernels:
 *   k_meth_bounds  one workgroup per 8192 pairs of one read (the tiles of a
 *                  bound of each read's path, from the host's offsets): the
 *                  first and last event paired with each k-mer (the pairs run
 *                  in path order, so a k-mer's pairs are consecutive);
 *   k_meth_sites   one workgroup per 8192 k-mers of one read: the sites
 *                  appended to a list (one atomic per workgroup), NaN / 0
 *                  written for every k-mer;
 *   k_meth_llr     one thread per listed site: both profiles in registers (a
 *                  column of at most ABEA_MAX_K cells per model), then the LLR.
 */
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "abea_internal.h"

namespace abea {

namespace {

constexpr int KMAX = 12; /* the longest window: k <= ABEA_MAX_K */
constexpr int CHUNK = METH_CHUNK; /* pairs or k-mers per workgroup of the first two kernels */

__device__ __forceinline__ bool is_site(uint32_t rank, int k) {
  return k >= 2 && ((rank >> (2 * (k - 1))) & 3u) == 1u && ((rank >> (2 * (k - 2))) & 3u) == 2u;
}

}  // namespace

/* the plan (reads and tile tables) from pinned host memory into device
 * memory, and the site counter zeroed: a kernel, so that nothing of the call
 * waits in the copy engines' queues behind another stream's work */
__global__ __launch_bounds__(256) void k_meth_stage(const uint64_t *src, uint64_t *dst, size_t words,
                                                    uint32_t *n_sites) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) *n_sites = 0u;
  if (i < words) dst[i] = src[i];
}

/* v of the lane below (above), and `edge` in lane 0 (63): DPP wave_shr:1, wave_shl:1 */
__device__ __forceinline__ int lane_below(int edge, int v) {
  return __builtin_amdgcn_update_dpp(edge, v, 0x138, 0xF, 0xF, false);
}
__device__ __forceinline__ int lane_above(int edge, int v) {
  return __builtin_amdgcn_update_dpp(edge, v, 0x130, 0xF, 0xF, false);
}

/* one workgroup per tile, a run of CHUNK pairs of one read, a quarter of it per
 * wavefront: the first and the last event paired with each k-mer (a k-mer's
 * pairs are consecutive in the path order).  The read's fields are
 * workgroup-uniform; the wavefront loads G * 64 consecutive pairs, once, and
 * takes a pair's neighbours from the lanes beside it (three loads per pair: 181
 * us for 4000 reads of 5 kb, this 153). */
__global__ __launch_bounds__(256) void k_meth_bounds(MethArgs a) {
  const MethTile tl = a.pair_tiles[blockIdx.x];
  const int r = (int)tl.read;
  if (a.status[r] != READ_OK) return;
  const uint64_t p0 = a.pair_offset[r], p1 = a.pair_offset[r + 1];
  const uint64_t c0 = p0 + (uint64_t)tl.chunk * CHUNK;
  if (c0 >= p1) return;
  const MethRead rd = a.reads[r];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr int G = 8, PER_WAVE = CHUNK / 4;
  for (int g = 0; g < PER_WAVE; g += G * 64) {
    const uint64_t pw = c0 + (uint64_t)(wave * PER_WAVE + g);
    if (pw >= p1) return;
    int2 q[G];
#pragma unroll
    for (int u = 0; u < G; ++u) {
      const uint64_t p = pw + (uint64_t)(64 * u + lane);
      q[u] = p < p1 ? a.pairs[p] : make_int2(0, -1);
    }
    /* the k-mers before and after the run (none: no k-mer's) */
    int edge = INT32_MIN;
    if (lane == 0 && pw > p0) edge = a.pairs[pw - 1].y;
    if (lane == 63 && pw + G * 64 < p1) edge = a.pairs[pw + G * 64].y;
#pragma unroll
    for (int u = 0; u < G; ++u) {
      const int y = q[u].y;
      const int yp = lane_below(u == 0 ? edge : __builtin_amdgcn_readlane(q[u > 0 ? u - 1 : 0].y, 63), y);
      const int yn = lane_above(u == G - 1 ? edge : __builtin_amdgcn_readlane(q[u < G - 1 ? u + 1 : u].y, 0), y);
      if (y < 0 || y >= rd.n_k) continue;
      if (yp != y) a.kfirst[rd.km_off + y] = q[u].x;
      if (yn != y) a.klast[rd.km_off + y] = q[u].x;
    }
  }
}

typedef uint32_t u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

/* one workgroup per tile, a run of CHUNK k-mers of one read, four consecutive per
 * thread and step: the sites of an aligned read go to the list (one atomic per
 * workgroup: the sites are found and counted first, four bits per step kept by
 * each thread, then written at the workgroup's base), and every k-mer gets NaN
 * and 0, which k_meth_llr replaces at the sites (a k-mer per thread and step: 118
 * us for 4000 reads of 5 kb, this 87) */
__global__ __launch_bounds__(256) void k_meth_sites(MethArgs a) {
  __shared__ uint32_t wcount[4], wbase[4];
  const MethTile tl = a.kmer_tiles[blockIdx.x];
  const int r = (int)tl.read;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const MethRead rd = a.reads[r];
  const bool ok = a.status[r] == READ_OK;
  const uint32_t j0 = tl.chunk * (uint32_t)CHUNK; /* the run's first k-mer in the read */
  const uint32_t nj = (uint32_t)rd.n_k - j0 < (uint32_t)CHUNK ? (uint32_t)rd.n_k - j0 : (uint32_t)CHUNK;
  constexpr int STEPS = CHUNK / 1024;
  static_assert(STEPS * 4 == 32, "a thread's sites in one word");
  const uint32_t *rank = a.ranks + rd.km_off + j0;
  float *llr = a.llr + rd.km_off + j0;
  int32_t *n_ev = a.n_ev ? a.n_ev + rd.km_off + j0 : nullptr;
  uint32_t bits = 0, cnt = 0;
#pragma unroll
  for (int it = 0; it < STEPS; ++it) {
    const uint32_t j = (uint32_t)(it * 1024) + 4u * threadIdx.x;
    uint32_t b = 0;
    if (j + 4 <= nj) {
      const u32x4_a4 k4 = *reinterpret_cast<const u32x4_a4 *>(rank + j);
#pragma unroll
      for (int u = 0; u < 4; ++u) b |= (uint32_t)is_site(k4[u], a.k) << u;
      *reinterpret_cast<f32x4_a4 *>(llr + j) = f32x4_a4{NAN, NAN, NAN, NAN};
      if (n_ev) *reinterpret_cast<u32x4_a4 *>(n_ev + j) = u32x4_a4{0, 0, 0, 0};
    } else {
      for (uint32_t u = 0; u < 4 && j + u < nj; ++u) {
        b |= (uint32_t)is_site(rank[j + u], a.k) << u;
        llr[j + u] = NAN;
        if (n_ev) n_ev[j + u] = 0;
      }
    }
    if (!ok) b = 0;
    bits |= b << (4 * it);
#pragma unroll
    for (int u = 0; u < 4; ++u) cnt += (uint32_t)__popcll(__ballot((b >> u) & 1u));
  }
  if (lane == 0) wcount[wave] = cnt;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t t = 0;
    for (int w = 0; w < 4; ++w) t += wcount[w];
    uint32_t b = t ? atomicAdd(a.n_sites, t) : 0u;
    for (int w = 0; w < 4; ++w) {
      wbase[w] = b;
      b += wcount[w];
    }
  }
  __syncthreads();
  uint32_t run = wbase[wave];
#pragma unroll
  for (int it = 0; it < STEPS; ++it) {
    const uint32_t b = (bits >> (4 * it)) & 15u;
    uint32_t slot = run;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint64_t m = __ballot((b >> u) & 1u);
      slot += (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
      run += (uint32_t)__popcll(m);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if ((b >> u) & 1u) a.sites[slot++] = make_uint2((uint32_t)r, j0 + (uint32_t)(it * 1024 + u) + 4u * threadIdx.x);
  }
}

/* One thread per site: both profiles' columns in registers.
 *
 * What bounds it: the gathers of a site (its k-mers, their entries of two models,
 * its events), each from a cache line of its own; most miss the L1, whose pending
 * lines then hold the others up (411 us for the 2 M sites of 4000 reads of 5 kb).
 * K, the longest window, is the context's k: registers for it alone, and AHEAD events
 * requested at once (375 us).  Up to k = 6 both models' tables (128 KB at most) lie in
 * LDS, with workgroups of LLR_LDS_THREADS: 301 us.  A window cut off by the read's
 * start is filled up in front with k-mers whose emission is -inf. */
constexpr int AHEAD = 4;
constexpr int LLR_LDS_THREADS = 1024;
template <int K>
struct LlrModels {
  static_assert(K >= 2 && K <= KMAX, "a site's window");
  static constexpr bool LDS = K <= 6;
  static constexpr int ENTRIES = LDS ? 1 << (2 * K) : 1;
  static constexpr int THREADS = LDS ? LLR_LDS_THREADS : 256;
  /* workgroups: as many as the device holds at once, by their threads two a CU, by
   * the tables' 128 KB of the CU's 160 one at k = 6; without tables 2048 */
  static int groups(int cus) { return !LDS ? 2048 : K == 6 ? cus : 2 * cus; }
};
static_assert(sizeof(ModelEntry) == sizeof(float4), "an entry is read as a float4");

template <int K>
__global__ __launch_bounds__(LlrModels<K>::THREADS) void k_meth_llr(MethArgs a) {
  constexpr bool LDS = LlrModels<K>::LDS;
  __shared__ float4 tab[LDS ? 2 : 1][LlrModels<K>::ENTRIES];
  const uint32_t n_sites = *a.n_sites;
  if (LDS) {
    if (blockIdx.x * blockDim.x >= n_sites) return;
    for (int j = threadIdx.x; j < LlrModels<K>::ENTRIES; j += LlrModels<K>::THREADS) {
      tab[0][j] = reinterpret_cast<const float4 *>(a.model)[j];
      tab[LDS ? 1 : 0][j] = reinterpret_cast<const float4 *>(a.meth_model)[j];
    }
    __syncthreads();
  }
  const float NI = -INFINITY;
  for (uint32_t s = blockIdx.x * blockDim.x + threadIdx.x; s < n_sites; s += gridDim.x * blockDim.x) {
    const uint2 st = a.sites[s];
    const MethRead rd = a.reads[st.x];
    const int32_t i = (int32_t)st.y;
    const int32_t j0 = i - (K - 1) > 0 ? i - (K - 1) : 0;
    const int first = K - (i - j0 + 1); /* the window's first k-mer among the K */
    const int32_t e0 = a.kfirst[rd.km_off + j0], e1 = a.klast[rd.km_off + i];
    const float scale = a.scale[st.x], shift = a.shift[st.x];
    const float *xm = a.events + (uint64_t)a.ev_stride * rd.ev_off;
    float xn[AHEAD];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) xn[u] = xm[(uint64_t)a.ev_stride * (uint64_t)min(e0 + u, max(e0, e1))];
    /* the window's k-mer parameters under both models */
    float mu_u[K], c_u[K], h_u[K], mu_m[K], c_m[K], h_m[K];
#pragma unroll
    for (int j = 0; j < K; ++j) {
      const uint32_t rk = a.ranks[rd.km_off + (uint64_t)(i - min(K - 1 - j, i - j0))];
      float4 u, m; /* mean, c, h */
      if (LDS) {
        u = tab[0][rk & (uint32_t)(LlrModels<K>::ENTRIES - 1)];
        m = tab[LDS ? 1 : 0][rk & (uint32_t)(LlrModels<K>::ENTRIES - 1)];
      } else {
        u = reinterpret_cast<const float4 *>(a.model)[rk];
        m = reinterpret_cast<const float4 *>(a.meth_model)[rk];
      }
      mu_u[j] = a.scale_events ? u.x : __builtin_fmaf(u.x, scale, shift);
      mu_m[j] = a.scale_events ? m.x : __builtin_fmaf(m.x, scale, shift);
      c_u[j] = j < first ? NI : u.y;
      h_u[j] = u.z;
      c_m[j] = j < first ? NI : m.y;
      h_m[j] = m.z;
    }
    /* columns of the previous event, su[j+1] k-mer j's: before the first event all
     * -inf but the origin, the diagonal neighbour of the first k-mer */
    float su[K + 1], sm[K + 1];
#pragma unroll
    for (int j = 0; j <= K; ++j) su[j] = sm[j] = j == first ? 0.0f : NI;
    /* the next AHEAD events' means are loaded while these ones' rows are computed */
    for (int32_t e = e0; e <= e1; e += AHEAD) {
      float xs[AHEAD];
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) xs[u] = xn[u];
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) xn[u] = xm[(uint64_t)a.ev_stride * (uint64_t)min(e + AHEAD + u, e1)];
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) {
        if (e + u > e1) break;
        float x = xs[u];
        if (a.scale_events) {
          const float d = x - shift;
          x = d / scale;
        }
        float du = su[0], dm = sm[0];
        float lu = NI, lm = NI; /* left neighbours in this event's row */
        su[0] = sm[0] = NI;
#pragma unroll
        for (int j = 0; j < K; ++j) {
          const float d_u = x - mu_u[j];
          const float em_u = c_u[j] - ((d_u * d_u) * h_u[j]);
          const float d_m = x - mu_m[j];
          const float em_m = c_m[j] - ((d_m * d_m) * h_m[j]);
          const float nu = fmaxf(fmaxf((du + rd.lp_step) + em_u, (su[j + 1] + rd.lp_stay) + em_u), lu + rd.lp_skip);
          const float nm = fmaxf(fmaxf((dm + rd.lp_step) + em_m, (sm[j + 1] + rd.lp_stay) + em_m), lm + rd.lp_skip);
          du = su[j + 1];
          dm = sm[j + 1];
          su[j + 1] = nu;
          sm[j + 1] = nm;
          lu = nu;
          lm = nm;
        }
      }
    }
    a.llr[rd.km_off + i] = sm[K] - su[K];
    if (a.n_ev) a.n_ev[rd.km_off + i] = e1 - e0 + 1;
  }
}

hipError_t launch_meth_stage(const uint64_t *src, uint64_t *dst, size_t words, uint32_t *n_sites, hipStream_t st) {
  const size_t blocks = (words + 255) / 256;
  hipLaunchKernelGGL(k_meth_stage, dim3((uint32_t)(blocks > 0 ? blocks : 1)), dim3(256), 0, st, src, dst, words,
                     n_sites);
  return hipGetLastError();
}

hipError_t launch_meth(const MethArgs &a, int cus, hipStream_t st, hipEvent_t *tev) {
  if (a.n_reads > 0 && a.n_kmers > 0) {
    if (a.n_pair_tiles > 0)
      hipExtLaunchKernelGGL(k_meth_bounds, dim3(a.n_pair_tiles), dim3(256), 0, st, tev ? tev[0] : nullptr, nullptr, 0,
                            a);
    else if (tev)
      (void)hipEventRecord(tev[0], st);
    hipExtLaunchKernelGGL(k_meth_sites, dim3(a.n_kmer_tiles), dim3(256), 0, st, nullptr, tev ? tev[1] : nullptr, 0,
                          a);
    hipEvent_t t0 = tev ? tev[2] : nullptr, t1 = tev ? tev[3] : nullptr;
    switch (a.k) {
#define ABEA_LLR(K)                                                                                                   \
  case K:                                                                                                             \
    hipExtLaunchKernelGGL(k_meth_llr<K>, dim3(LlrModels<K>::groups(cus)), dim3(LlrModels<K>::THREADS), 0, st, t0, t1, \
                          0, a);                                                                                      \
    break;
      case 1: /* (no site) */
      ABEA_LLR(2)
      ABEA_LLR(3)
      ABEA_LLR(4)
      ABEA_LLR(5)
      ABEA_LLR(6)
      ABEA_LLR(7)
      ABEA_LLR(8)
      ABEA_LLR(9)
      ABEA_LLR(10)
      ABEA_LLR(11)
      ABEA_LLR(12)
#undef ABEA_LLR
      default: return hipErrorInvalidValue;
    }
  }
  return hipGetLastError();
}

}  // namespace abea
