/*
 * abea_detect.hip -- gfx950 kernels of event detection: the segmentation of
 * each read's raw signal into events {mean, stdv, n} at sudden changes of the
 * signal level (the thesis, Ch. 5 §5.2.2 "Methylation calling", its
 * event-detection paragraph; its output is the event table of Alg. 5.1).
 *
 * The thesis gives no algorithm for the step.  The detector is a two-window
 * change-point test:
 *   - at a boundary i (between samples i-1 and i; defined for
 *     w <= i <= n-w) the squared two-sample t statistic of the w samples
 *     before and the w after, with population variances, is w D^2 / V with
 *     D = S_r - S_l and V = w (Q_l + Q_r) - S_l^2 - S_r^2 (S sums, Q sums of
 *     squares: exact integers); the quotient is taken in float32 as
 *     ((float)D * (float)D) * (float)w / (float)(double)V, +inf for V = 0 and
 *     D != 0, 0 for V = 0 and D = 0;
 *   - i is a peak of the detector (w, t) if its statistic exceeds t^2 (as a
 *     float), is greater than the statistic at every defined boundary up to
 *     w-1 before it and not less than at every one up to w-1 after it;
 *   - a short and a long detector; every peak of either starts an event;
 *   - an event's mean and stdv come from its exact integer sum S and sum of
 *     squares Q: m = (double)S / len, V = len*Q - S^2 (exact, then rounded
 *     once to double), mean = (float)((m + offset) * pa_scale),
 *     stdv = (float)(sqrt(V) / len * pa_scale), pA = (raw + offset) * pa_scale.
 *
 * The work is a stream over the raw samples:
 *   k_ed_tiles     the tile table (one wavefront per read);
 *   k_ed_detect    one wavefront per tile of 1024 boundaries of one read: both
 *                  statistics, peaks, one bit per boundary, and the tile's
 *                  event count and first change point (k_ed_detect_any, a
 *                  workgroup per tile, for windows other than 3 and 8);
 *   k_ed_scan      exclusive scan of the tile counts, per 1024 tiles, then
 *                  over the blocks (k_ed_scan_top); with one block and no
 *                  more reads than it has tiles, also k_ed_offsets' work;
 *   k_ed_events    one wavefront per tile: the tile's event starts in order,
 *                  the end of its last event from the first change point of
 *                  the read's next tiles, and one lane per event for its
 *                  statistics;
 *   k_ed_offsets   each read's first event.
 */
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "abea_internal.h"

namespace abea {

namespace {

constexpr int TS = ED_TILE;   /* boundaries per tile */
constexpr int WMAX = ED_MAX_WINDOW;
constexpr int XH = 2 * WMAX;  /* samples kept before (and after) the tile */
constexpr int THL = WMAX;     /* statistics kept before (and after) the tile */
constexpr int NX = TS + 2 * XH;
constexpr int NT = TS + 2 * THL;
constexpr int WORDS = TS / 64; /* flag words per tile */
constexpr int THREADS = 256;
constexpr int SCAN_TILES = 1024; /* tiles per block of the first scan level */

/* a / b rounded to nearest, for 0 <= a < 2^64 and 1 <= b < 2^64: a
 * reciprocal estimate refined by one Newton step, a first quotient, and two
 * corrections from exact residuals (FMA).  It is the refinement the general
 * FP32 division performs; the general one also scales operands whose
 * quotient or reciprocal would leave the normal range and patches zero,
 * infinite and NaN operands, none of which arises here (a = 0 gives +0). */
__device__ __forceinline__ float div_small(float a, float b) {
  float y0; /* the reciprocal starts alone: raised priority, see k_ed_detect */
  asm("s_setprio 1\n\tv_rcp_f32 %0, %1\n\ts_setprio 0\n\ts_nop 0" : "=v"(y0) : "v"(b));
  const float e = __builtin_fmaf(-b, y0, 1.0f);
  const float y = __builtin_fmaf(e, y0, y0);
  const float q0 = a * y;
  const float r0 = __builtin_fmaf(-b, q0, a);
  const float q1 = __builtin_fmaf(r0, y, q0);
  const float r1 = __builtin_fmaf(-b, q1, a);
  return __builtin_fmaf(r1, y, q1);
}

/* statistic of the detector with window w at boundary j of a read of n
 * samples, from prefix sums: P[c] and PQ[c] sum the staged samples before
 * sample j (and their squares).  Q_l + Q_r and V are taken in double, where
 * every value is an integer below 2^41 (at most 2 * 16 * 2^30 for the sums of
 * squares, 2^40 for w (Q_l + Q_r) and S^2), so each operation is exact and V
 * is the exact integer.  Branch-free: the loads stay inside the staged range
 * for every boundary of the tile and its halo. */
__device__ __forceinline__ float ed_stat(const int *P, const double *PQ, int c, int w, int j, int n) {
  const int sl = P[c] - P[c - w];
  const int sr = P[c + w] - P[c];
  const double q = PQ[c + w] - PQ[c - w];
  const double dl = (double)sl, dr = (double)sr;
  const double v = __builtin_fma(-dl, dl, __builtin_fma(-dr, dr, (double)w * q));
  const int d = sr - sl;
  const float df = (float)d;
  const float num = (df * df) * (float)w;
  const float den = (float)v;
  const float qt = div_small(num, v == 0.0 ? 1.0f : den);
  const float t = v != 0.0 ? qt : (d != 0 ? INFINITY : 0.0f);
  return (j >= w && j <= n - w) ? t : -1.0f;
}

/* per lane: the larger of a and b, and the largest of a, b and c (one
 * v_max_f32 / v_max3_f32 without canonicalisation: the statistics are never
 * NaN) */
__device__ __forceinline__ float max2(float a, float b) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ float max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

/* Peaks of the detector (window w, thr = t^2) at the four boundaries
 * ts[q0 .. q0+3]: boundary q is a peak if ts[q] is above thr and above every
 * statistic up to w-1 before it, and not below any up to w-1 after it.
 * Undefined boundaries hold -1, below every defined statistic, so they never
 * block a peak; thr >= 0 takes part in the maximum before (t > thr and
 * t > max(before) is t > max(thr, before)). */
__device__ __forceinline__ uint32_t ed_peaks4(const float *ts, int q0, int w, float thr) {
  uint32_t bits = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int q = q0 + j;
    const float t = ts[q];
    float lm = thr, rm = -1.0f;
    for (int m = 1; m < w; ++m) {
      lm = fmaxf(lm, ts[q - m]);
      rm = fmaxf(rm, ts[q + m]);
    }
    bits |= ((t > lm) & (t >= rm)) ? (1u << j) : 0u;
  }
  return bits;
}

/* between LDS writes and reads by other lanes of the same wavefront: its accesses
 * execute in order, and the compiler keeps them in order */
__device__ __forceinline__ void wave_exchange() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

/* v of lane l-n of the same row of 16 lanes, cyclically (DPP row_ror:n) */
template <int N>
__device__ __forceinline__ uint32_t row_ror(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x120 + N, 0xF, 0xF, true);
}

/* Stage samples base+k, k in [0, NS), of a read (zero outside [0, lim)) as
 * prefix sums: P[k] and PQ[k] sum the first k values and their squares
 * (QT: long long, or double, exact for NS * 2^30 < 2^53).
 * Thread t takes PER_ consecutive samples; the sums are scanned over the wave
 * and over the waves.  Ends with a barrier. */
/* inclusive scan over the 64 lanes of a wavefront by DPP: within each row
 * of 16 lanes by shifts of 1, 2, 4 and 8 (lanes without a source add 0),
 * then lane 15 of each row into the next row and lane 31 into the upper
 * half */
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_i(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xF, true);
}
__device__ __forceinline__ int wave_scan(int v) {
  v += dpp_i<0x111, 0xF>(v); /* row_shr:1 */
  v += dpp_i<0x112, 0xF>(v); /* row_shr:2 */
  v += dpp_i<0x114, 0xF>(v); /* row_shr:4 */
  v += dpp_i<0x118, 0xF>(v); /* row_shr:8 */
  v += dpp_i<0x142, 0xA>(v); /* row_bcast:15 into rows 1 and 3 */
  v += dpp_i<0x143, 0xC>(v); /* row_bcast:31 into rows 2 and 3 */
  return v;
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_d(double v) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)dpp_i<CTRL, ROWS>((int)(uint32_t)b);
  const uint32_t hi = (uint32_t)dpp_i<CTRL, ROWS>((int)(uint32_t)(b >> 32));
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
/* the same over 64-bit integers, and over doubles that hold integers below
 * 2^53 (every sum exact) */
__device__ __forceinline__ double wave_scan(double v) {
  v += dpp_d<0x111, 0xF>(v);
  v += dpp_d<0x112, 0xF>(v);
  v += dpp_d<0x114, 0xF>(v);
  v += dpp_d<0x118, 0xF>(v);
  v += dpp_d<0x142, 0xA>(v);
  v += dpp_d<0x143, 0xC>(v);
  return v;
}
template <int CTRL, int ROWS>
__device__ __forceinline__ long long dpp_l(long long v) {
  const uint64_t b = (uint64_t)v;
  const uint32_t lo = (uint32_t)dpp_i<CTRL, ROWS>((int)(uint32_t)b);
  const uint32_t hi = (uint32_t)dpp_i<CTRL, ROWS>((int)(uint32_t)(b >> 32));
  return (long long)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ long long wave_scan(long long v) {
  v += dpp_l<0x111, 0xF>(v);
  v += dpp_l<0x112, 0xF>(v);
  v += dpp_l<0x114, 0xF>(v);
  v += dpp_l<0x118, 0xF>(v);
  v += dpp_l<0x142, 0xA>(v);
  v += dpp_l<0x143, 0xC>(v);
  return v;
}

__device__ __forceinline__ long long last_lane(long long v) {
  return (long long)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), 63) << 32) |
                     (uint32_t)__builtin_amdgcn_readlane((int)v, 63));
}

template <int NS, typename QT>
__device__ __forceinline__ void stage_prefix(const int16_t *x, int64_t base, int64_t lim, int *P, QT *PQ, int *wsum,
                                             QT *wsq) {
  constexpr int PER_ = (NS + THREADS - 1) / THREADS;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int v[PER_];
  int s = 0;
  QT q = 0;
#pragma unroll
  for (int e = 0; e < PER_; ++e) {
    const int k = PER_ * (int)threadIdx.x + e;
    const int64_t si = base + k;
    v[e] = (k < NS && si >= 0 && si < lim) ? (int)x[si] : 0;
    s += v[e];
    q += (QT)(v[e] * v[e]);
  }
  const int si = wave_scan(s);
  const QT qi = wave_scan(q);
  if (lane == 63) {
    wsum[wave] = si;
    wsq[wave] = qi;
  }
  __syncthreads();
  int ps = si - s;
  QT pq = qi - q;
  for (int w = 0; w < wave; ++w) {
    ps += wsum[w];
    pq += wsq[w];
  }
  if (threadIdx.x == 0) {
    P[0] = 0;
    PQ[0] = 0;
  }
#pragma unroll
  for (int e = 0; e < PER_; ++e) {
    const int k = PER_ * (int)threadIdx.x + e;
    ps += v[e];
    pq += (QT)(v[e] * v[e]);
    if (k < NS) {
      P[k + 1] = ps;
      PQ[k + 1] = pq;
    }
  }
  __syncthreads();
}

}  // namespace

/* the tile table: one wavefront per read writes its tiles' entries */
__global__ void k_ed_tiles(DetectArgs a) {
  const int r = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (r >= a.n_reads) return;
  const uint64_t s0 = a.sample_offset[r];
  const uint32_t n = (uint32_t)(a.sample_offset[r + 1] - s0);
  const uint32_t t0 = a.tile_first[r], t1 = a.tile_first[r + 1];
  for (uint32_t t = t0 + (threadIdx.x & 63); t < t1; t += 64) {
    EdTile e;
    e.s0 = s0;
    e.n = n;
    e.i0 = (t - t0) * (uint32_t)TS;
    e.read = (uint32_t)r;
    e.g_end = t1;
    a.tiles[t] = e;
  }
}

/* ------------------------------------- change points, windows of 3 and 8 */

/* The default windows, known at compile time: a wavefront takes a tile, a lane
 * 16 consecutive boundaries of it.
 *
 * What bounds it: the vector instructions of the two statistics (about 1200 per
 * lane for 16 boundaries); the samples are read once and a tile's results are
 * 128 bytes.  Two wavefronts of a SIMD start simple float instructions side by
 * side, but double-precision operations, of which a thread that takes the
 * statistics from prefix sums in LDS runs 6 each, and 24-bit multiplications only
 * alone: 291 M samples (4000 reads of 5 kb) take 966 us in that form, 625 in
 * exact 32-bit integers and 460 in this.  The reciprocals, which start alone too,
 * run at raised priority, so that the wavefronts at one pass it first and the
 * others find partners (513 us without).  A lane keeps
 * its 16 + 2 * 8 samples as float32 in registers, and its window sums slide.  D and
 * V are differences, the same integers for samples less a constant: with a constant
 * near the lane's mean the sum of any 24 squares lies below 2^21 in any usual
 * signal (a deviation of 295 all along), and then every sum, square and V is an
 * integer below 2^24 (w (Q_l + Q_r) <= 8 * 2^21, and S_l^2 + S_r^2 is no larger),
 * exact at each step.  A tile in which some lane's sum is larger takes
 * wide_stats.  The roundings of the statistic's operands and its quotient are as
 * in ed_stat. */
constexpr int BPL = 16;          /* boundaries per lane */
constexpr int HB = 8;            /* boundaries (and samples) looked at beyond a lane's or the tile's */
constexpr int ROW = (64 + 2) * (BPL + 4); /* floats: lane l's statistics at (l+1) * 20, 16-byte pieces of 16 lanes in different banks */
constexpr float MAX_SQUARES = 2097152.0f; /* of the 16 samples around a boundary, below which all is exact */
static_assert(TS == 64 * BPL, "a wavefront per tile");

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
/* words at any sample's address */
typedef u32x4 u32x4_a2 __attribute__((aligned(2)));
typedef uint32_t u32_a2 __attribute__((aligned(2)));
static_assert(alignof(u32x4_a2) == alignof(int16_t) && alignof(u32_a2) == alignof(int16_t),
              "loads of words promise no more than a sample's alignment");

/* A tile's read as seen from the tile's first boundary: samples at x[lo .. hi],
 * boundaries of a window w defined in [w - first, last - w] (32 bits, cut off
 * beyond the tile's reach). */
struct TileView {
  const int16_t *x;
  int lo, hi;
  int odd;     /* 1: x lies two bytes after a multiple of four */
  bool inside; /* every sample within 2 * HB + 2 of the tile is the read's */
};

__device__ __forceinline__ TileView tile_view(const int16_t *x, int64_t i0, int64_t n) {
  TileView v;
  v.x = x + i0;
  v.lo = i0 < 64 ? -(int)i0 : -64;
  v.hi = n - 1 - i0 < 4096 ? (int)(n - 1 - i0) : 4096;
  v.odd = (int)(reinterpret_cast<uintptr_t>(v.x) >> 1) & 1;
  v.inside = v.lo <= -2 * HB - 2 && v.hi >= TS + 2 * HB + 1;
  return v;
}

__device__ __forceinline__ int sample_at(const TileView &v, int rel) {
  return v.x[min(max(rel, v.lo), v.hi)];
}

/* samples rel .. rel + 2*NW - 1 of the read as pairs.  A read's samples start at
 * any even address: for even rel (the lanes' own boundaries) the words are read
 * from multiples of four bytes, for odd rel (half of the halo boundaries) from two
 * bytes after one, in both cases from as much as a sample before rel to two
 * after the last. */
template <int NW>
__device__ __forceinline__ void word_pairs(const TileView &v, int rel, uint32_t (&d)[NW]) {
  const u32x4_a2 *p = reinterpret_cast<const u32x4_a2 *>(v.x + rel - v.odd);
#pragma unroll
  for (int i = 0; i < NW / 4; ++i) {
    const u32x4 q = p[i];
    d[4 * i] = q.x;
    d[4 * i + 1] = q.y;
    d[4 * i + 2] = q.z;
    d[4 * i + 3] = q.w;
  }
  if (v.odd) {
    const uint32_t e = reinterpret_cast<const u32_a2 *>(p)[NW];
#pragma unroll
    for (int i = 0; i < NW; ++i) d[i] = __builtin_amdgcn_alignbit(i + 1 < NW ? d[i + 1] : e, d[i], 16);
  }
}

/* the same near the read's ends (outside it: its nearest sample; no defined
 * boundary reaches one) */
template <int NW>
__device__ __forceinline__ void sample_pairs(const TileView &v, int rel, uint32_t (&d)[NW]) {
  if (v.inside) {
    word_pairs(v, rel, d);
  } else {
#pragma unroll
    for (int i = 0; i < NW; ++i)
      d[i] = ((uint32_t)sample_at(v, rel + 2 * i) & 0xffffu) | ((uint32_t)sample_at(v, rel + 2 * i + 1) << 16);
  }
}

/* a constant in a vector register: an instruction with a scalar or literal
 * operand takes the place of two with vector operands */
template <typename T>
__device__ __forceinline__ T vreg(T c) {
  T r;
  asm("v_mov_b32 %0, %1" : "=v"(r) : "i"(c));
  return r;
}
struct Consts {
  uint32_t low, mag;
  float tiny;
};
__device__ __forceinline__ Consts consts() {
  return {vreg(0xffffu), vreg(0x4b008000u), __uint_as_float(vreg(0x1f800000u) /* 2^-64 */)};
}

/* 2*NW samples (pairs) less an integer near their mean, as floats: a sample plus
 * 2^15 is put into the mantissa of 2^23, and differences of such floats are
 * exact. */
template <int NW>
__device__ __forceinline__ void centred(const Consts &k, const uint32_t (&d)[NW], float (&y)[2 * NW]) {
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    y[2 * i] = __uint_as_float(__builtin_amdgcn_bitop3_b32(d[i], k.low, k.mag, 0x6a)); /* (d & low) ^ mag */
    uint32_t high; /* (the compiler would take the half in the xor, an SDWA instruction, which starts alone) */
    asm("v_lshrrev_b32 %0, 16, %1" : "=v"(high) : "v"(d[i]));
    y[2 * i + 1] = __uint_as_float(high ^ k.mag);
  }
  /* four floats of [2^23, 2^24): their sum is a multiple of 4 */
  const float c = ((y[NW / 4] + y[3 * NW / 4]) + (y[5 * NW / 4] + y[7 * NW / 4])) * 0.25f;
#pragma unroll
  for (int i = 0; i < 2 * NW; ++i) y[i] -= c;
}

/* The statistic of a window w from D and V (both exact), kept between the
 * threshold and T_INF.  It stands for infinity: where V = 0 (V + 2^-64 is V
 * otherwise) the quotient num / 2^-64 (num is 0 or 4 to 2^41) is 0 or beyond it,
 * and no other statistic reaches 2^42.  Peaks depend on the order of statistics
 * alone, and on that of none below the threshold. */
constexpr float T_INF = 0x1p60f;
__device__ __forceinline__ float kept_stat(const Consts &k, float w, float df, float v, float thr) {
  const float num = (df * df) * w;
  return __builtin_amdgcn_fmed3f(div_small(num, v + k.tiny), thr, T_INF);
}

/* the same from the window sums and the sum of squares over both windows */
__device__ __forceinline__ float stat_f32(const Consts &k, float w, float sl, float sr, float q, float thr) {
  return kept_stat(k, w, sr - sl, __builtin_fmaf(-sl, sl, __builtin_fmaf(-sr, sr, w * q)), thr);
}

/* The kept statistics of window W at N consecutive boundaries, the first with HB
 * samples (pairs) before it, from any samples: sums in 32 bits, squares and V in
 * double, all exact. */
template <int W, int N, int NW>
__device__ __forceinline__ void wide_stats(const Consts &ks, const uint32_t (&d)[NW], float thr, float (&t)[N]) {
  static_assert(2 * NW >= N - 1 + 2 * HB, "samples on either side of each boundary");
  auto x = [&](int k) { return (k & 1) ? (int)d[k / 2] >> 16 : (int)(int16_t)d[k / 2]; };
  int sl = 0, sr = 0;
  double q2 = 0.0;
#pragma unroll
  for (int k = HB - W; k < HB; ++k) {
    sl += x(k);
    sr += x(k + W);
    q2 += (double)(x(k) * x(k)) + (double)(x(k + W) * x(k + W));
  }
#pragma unroll
  for (int q = 0; q < N; ++q) {
    const double l = (double)sl, r = (double)sr;
    const double v = __builtin_fma(-l, l, __builtin_fma(-r, r, (double)W * q2));
    t[q] = kept_stat(ks, (float)W, (float)(sr - sl), (float)v, thr);
    if (q + 1 < N) {
      const int a = x(q + HB - W), b = x(q + HB), c = x(q + HB + W);
      sl += b - a;
      sr += c - b;
      q2 += (double)(c * c) - (double)(a * a);
    }
  }
}

/* The peaks of window W (see ed_peaks4) at the lane's boundaries, one bit each,
 * from the row of statistics, none below the threshold (raising a statistic
 * to it changes no peak).  Windows of neighbours share their maxima. */
template <int W>
__device__ __forceinline__ uint32_t row_peaks(const float *row) {
  constexpr int H = W - 1;
  const int lane = threadIdx.x & 63;
  float e[HB + BPL + HB]; /* boundaries -HB .. BPL + HB - 1 of the lane */
  const float *own = row + (lane + 1) * (BPL + 4);
#pragma unroll
  for (int f = 0; f < (HB + BPL + HB) / 4; ++f) {
    const int k = 4 * f - HB;
    const float *p = k < 0 ? own - (BPL + 4) + BPL + k : k < BPL ? own + k : own + (BPL + 4) + k - BPL;
    const float4 t = *reinterpret_cast<const float4 *>(p);
    e[4 * f] = t.x;
    e[4 * f + 1] = t.y;
    e[4 * f + 2] = t.z;
    e[4 * f + 3] = t.w;
  }
  float m[HB + BPL + HB]; /* m[i]: the largest of e[i .. i+H-1] */
  if constexpr (H == 2) {
#pragma unroll
    for (int i = HB - H; i <= HB + BPL; ++i) m[i] = max2(e[i], e[i + 1]);
  } else {
    static_assert(H == 7, "windows of 3 and 8");
    float m3[HB + BPL + HB];
#pragma unroll
    for (int i = HB - H; i <= HB + BPL + H - 3; ++i) m3[i] = max3(e[i], e[i + 1], e[i + 2]);
#pragma unroll
    for (int i = HB - H; i <= HB + BPL; ++i) m[i] = max3(m3[i], m3[i + 3], e[i + 6]);
  }
  uint32_t bits = 0;
#pragma unroll
  for (int q = 0; q < BPL; ++q)
    bits |= ((e[HB + q] > m[HB + q - H]) & (e[HB + q] >= m[HB + q + 1])) ? (1u << q) : 0u;
  return bits;
}

__device__ __forceinline__ void put_row(float *row, const float (&t)[BPL], float *halo, float h) {
  float4 *own = reinterpret_cast<float4 *>(row + ((threadIdx.x & 63) + 1) * (BPL + 4));
#pragma unroll
  for (int f = 0; f < BPL / 4; ++f) own[f] = make_float4(t[4 * f], t[4 * f + 1], t[4 * f + 2], t[4 * f + 3]);
  if ((threadIdx.x & 63) < 2 * HB) *halo = h;
}

__global__ __launch_bounds__(THREADS, 4) void k_ed_detect(DetectArgs a) {
  constexpr int WS = 3, WL = 8;
  /* thresholds as kept_stat orders them: above every finite statistic, but below
   * infinity unless infinite themselves */
  const float thr_s = a.thr_short == INFINITY ? T_INF : fminf(a.thr_short, 0.5f * T_INF);
  const float thr_l = a.thr_long == INFINITY ? T_INF : fminf(a.thr_long, 0.5f * T_INF);
  __shared__ __align__(16) float rows[THREADS / 64][ROW];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t g = blockIdx.x * (THREADS / 64) + wave;
  if (g >= a.n_tiles) return;
  float *row = rows[wave];
  const EdTile tl = a.tiles[g];
  const int64_t n = tl.n, i0 = tl.i0;
  const TileView tv = tile_view(a.raw + tl.s0, i0, n);
  /* the halo boundary of lanes 0 to 15 (HB before the tile, HB after it), and its place in the row */
  const int hq = lane & (2 * HB - 1);
  const int halo_rel = hq < HB ? hq - HB : TS + hq - HB;
  float *halo = row + (hq < HB ? BPL - HB + hq : 65 * (BPL + 4) + hq - HB);

  uint32_t d[BPL], h[HB]; /* samples around the lane's boundaries, and around its halo boundary */
  sample_pairs(tv, BPL * lane - HB, d);
  sample_pairs(tv, halo_rel - HB, h);
  /* the first and last defined boundary of the two windows */
  const int last = n - i0 < 8192 ? (int)(n - i0) : 8192;
  const int first = i0 < 64 ? (int)i0 : 64;
  /* boundary rel of window w is defined */
  auto defined = [&](int rel, int w) { return rel >= w - first && rel <= last - w; };

  float y[2 * BPL], u[2 * HB];
  const Consts ks = consts();
  centred(ks, d, y);
  centred(ks, h, u);
  const float w8 = __uint_as_float(vreg(0x41000000u)), w3 = __uint_as_float(vreg(0x40400000u));
  float t[BPL], th;
  bool ok;
  { /* the long window: y[q .. q+7] and y[q+8 .. q+15] around boundary q */
    float df[2 * BPL - WL], sl = 0.0f, sr = 0.0f, q2 = 0.0f;
#pragma unroll
    for (int k = 0; k < 2 * BPL - WL; ++k) df[k] = y[k + WL] - y[k];
#pragma unroll
    for (int k = 0; k < WL; ++k) {
      sl += y[k];
      sr += y[k + WL];
    }
#pragma unroll
    for (int k = 0; k < 2 * WL; ++k) q2 = __builtin_fmaf(y[k], y[k], q2);
    const float q0 = q2;
    float q8 = 0.0f;
#pragma unroll
    for (int q = 0; q < BPL; ++q) {
      if (q == BPL / 2) q8 = q2;
      t[q] = stat_f32(ks, w8, sl, sr, q2, thr_l);
      sl += df[q];
      if (q + WL < 2 * BPL - WL) sr += df[q + WL];
      q2 = __builtin_fmaf(y[q + 2 * WL], y[q + 2 * WL], __builtin_fmaf(-y[q], y[q], q2));
    }
    /* the 16 squares around a boundary are among those of two of these sums */
    ok = (q0 + q8 < MAX_SQUARES) & (q8 + q2 < MAX_SQUARES);
    sl = sr = q2 = 0.0f;
#pragma unroll
    for (int k = 0; k < HB; ++k) {
      sl += u[k];
      sr += u[k + HB];
      q2 = __builtin_fmaf(u[k + HB], u[k + HB], __builtin_fmaf(u[k], u[k], q2));
    }
    ok &= q2 < MAX_SQUARES;
    th = stat_f32(ks, w8, sl, sr, q2, thr_l);
  }
  /* the long window's sums hold the short one's samples */
  const bool wide = __ballot(!ok) != 0;
  if (wide) {
    float w[1];
    sample_pairs(tv, BPL * lane - HB, d);
    sample_pairs(tv, halo_rel - HB, h);
    wide_stats<WL>(ks, d, thr_l, t);
    wide_stats<WL>(ks, h, thr_l, w);
    th = w[0];
  }
  if (!tv.inside) {
#pragma unroll
    for (int q = 0; q < BPL; ++q) t[q] = defined(BPL * lane + q, WL) ? t[q] : thr_l;
    th = defined(halo_rel, WL) ? th : thr_l;
  }
  put_row(row, t, halo, th);
  __builtin_amdgcn_sched_barrier(0); /* the two windows' registers are not needed at once */
  { /* the short window */
    float s3[BPL + WS], q2 = 0.0f; /* s3[k]: the sum of the window that ends before boundary k */
#pragma unroll
    for (int k = 0; k < BPL + WS; ++k) s3[k] = (y[k + HB - 3] + y[k + HB - 2]) + y[k + HB - 1];
#pragma unroll
    for (int k = HB - WS; k < HB + WS; ++k) q2 = __builtin_fmaf(y[k], y[k], q2);
#pragma unroll
    for (int q = 0; q < BPL; ++q) {
      t[q] = stat_f32(ks, w3, s3[q], s3[q + WS], q2, thr_s);
      q2 = __builtin_fmaf(y[q + HB + WS], y[q + HB + WS], __builtin_fmaf(-y[q + HB - WS], y[q + HB - WS], q2));
    }
    q2 = 0.0f;
#pragma unroll
    for (int k = HB - WS; k < HB + WS; ++k) q2 = __builtin_fmaf(u[k], u[k], q2);
    th = stat_f32(ks, w3, (u[HB - 3] + u[HB - 2]) + u[HB - 1], (u[HB] + u[HB + 1]) + u[HB + 2], q2, thr_s);
  }
  if (wide) {
    float w[1];
    sample_pairs(tv, BPL * lane - HB, d);
    sample_pairs(tv, halo_rel - HB, h);
    wide_stats<WS>(ks, d, thr_s, t);
    wide_stats<WS>(ks, h, thr_s, w);
    th = w[0];
  }
  if (!tv.inside) {
#pragma unroll
    for (int q = 0; q < BPL; ++q) t[q] = defined(BPL * lane + q, WS) ? t[q] : thr_s;
    th = defined(halo_rel, WS) ? th : thr_s;
  }
  __builtin_amdgcn_sched_barrier(0);
  /* a wavefront's LDS accesses are in order: one row serves both windows */
  wave_exchange();
  uint32_t bits = row_peaks<WL>(row);
  wave_exchange();
  put_row(row, t, halo, th);
  wave_exchange();
  bits |= row_peaks<WS>(row);

  reinterpret_cast<uint16_t *>(a.flags + (uint64_t)g * WORDS)[lane] = (uint16_t)bits;
  const uint32_t count = (uint32_t)__builtin_amdgcn_readlane(wave_scan((int)__popc(bits)), 63);
  const uint64_t any = __ballot(bits != 0);
  int cp = -1;
  if (any) {
    const int l = __builtin_ctzll(any);
    cp = (int)(uint32_t)i0 + BPL * l + __builtin_ctz((uint32_t)__builtin_amdgcn_readlane((int)bits, l));
  }
  if (lane == 0) {
    a.count[g] = count + (i0 == 0 ? 1u : 0u); /* the read's first event starts at sample 0 */
    a.first_cp[g] = cp;                         /* the tile's first change point in the read, -1 if it has none */
  }
}

/* ------------------------------------------- change points, other windows */

/* One workgroup per tile, windows at run time. */
__global__ __launch_bounds__(THREADS) void k_ed_detect_any(DetectArgs a) {
  /* the prefix sums, then (once every thread holds its statistics in
   * registers) the two rows of statistics in the same bytes: a smaller LDS
   * footprint, more workgroups per CU */
  __shared__ __align__(16) unsigned char lds[(NX + 1) * (sizeof(double) + sizeof(int))];
  double *PQ = reinterpret_cast<double *>(lds);
  int *P = reinterpret_cast<int *>(lds + (NX + 1) * sizeof(double));
  float *tsh = reinterpret_cast<float *>(lds);
  float *tlg = tsh + NT;
  static_assert(2 * NT * sizeof(float) <= sizeof(lds) && (NT * sizeof(float)) % 16 == 0, "statistics fit");
  __shared__ int wsum[THREADS / 64];
  __shared__ double wsq[THREADS / 64];
  __shared__ uint32_t wcnt[THREADS / 64];
  __shared__ int32_t wfirst[THREADS / 64];
  static_assert(TS == 4 * THREADS, "four boundaries per thread");
  static_assert(THL == WMAX && THL % 4 == 0, "the peak loads stay inside the statistics");
  const uint32_t g = blockIdx.x;
  const EdTile tl = a.tiles[g];
  const int64_t n = tl.n;
  const int64_t i0 = tl.i0;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ws = a.w_short, wl = a.w_long;

  /* samples i0-XH .. i0+TS+XH-1 */
  stage_prefix<NX>(a.raw + tl.s0, i0 - XH, n, P, PQ, wsum, wsq);
  /* boundary j = i0 - THL + k: the sums before it are P[k + XH - THL] */
  /* j in 32 bits: reads hold fewer than 2^31 samples, so n - w fits, and a
   * j of 2^31 or more (past the read's end) wraps to a negative value, which
   * is outside [w, n - w] like j itself */
  constexpr int NIT = (NT + THREADS - 1) / THREADS;
  float rs[NIT], rl[NIT];
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int k = (int)threadIdx.x + THREADS * it;
    if (k < NT) {
      const int j = (int)((uint32_t)i0 - (uint32_t)THL + (uint32_t)k);
      const int c = k + XH - THL;
      rs[it] = ed_stat(P, PQ, c, ws, j, (int)n);
      rl[it] = ed_stat(P, PQ, c, wl, j, (int)n);
    }
  }
  __syncthreads(); /* every thread is done with the prefix sums */
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int k = (int)threadIdx.x + THREADS * it;
    if (k < NT) {
      tsh[k] = rs[it];
      tlg[k] = rl[it];
    }
  }
  __syncthreads();
  /* thread t: boundaries 4t .. 4t+3 of the tile (statistics q0 .. q0+3);
   * the neighbours read lie in q0-16 .. q0+19, inside [0, NT) */
  const int q0 = 4 * (int)threadIdx.x + THL;
  const uint32_t nib = ed_peaks4(tsh, q0, ws, a.thr_short) | ed_peaks4(tlg, q0, wl, a.thr_long);
  /* flag word m of the wave (its boundaries 64m .. 64m+63) is lanes 16m ..
   * 16m+15, four bits each: its low half from the row's lanes 0-7, its high
   * half from lanes 8-15, gathered by three row rotations (lane 7 and lane
   * 15 of the row end with the halves) */
  uint32_t x = nib << (4 * (lane & 7));
  x |= row_ror<1>(x);
  x |= row_ror<2>(x);
  x |= row_ror<4>(x);
  if ((lane & 7) == 7) {
    uint32_t *f32 = reinterpret_cast<uint32_t *>(a.flags + (uint64_t)g * WORDS + 4 * wave);
    f32[lane >> 3] = x;
  }
  /* the wave's change points and its first one (wave-uniform masks) */
  const uint64_t b0 = __ballot(nib & 1u), b1 = __ballot(nib & 2u), b2 = __ballot(nib & 4u), b3 = __ballot(nib & 8u);
  if (lane == 0) {
    wcnt[wave] = (uint32_t)(__popcll(b0) + __popcll(b1) + __popcll(b2) + __popcll(b3));
    const uint64_t any = b0 | b1 | b2 | b3;
    int32_t f = INT32_MAX;
    if (any) {
      const int l = __builtin_ctzll(any);
      const int j = ((b0 >> l) & 1u) ? 0 : ((b1 >> l) & 1u) ? 1 : ((b2 >> l) & 1u) ? 2 : 3;
      f = 256 * wave + 4 * l + j;
    }
    wfirst[wave] = f;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t c = (i0 == 0) ? 1u : 0u; /* the read's first event starts at sample 0 */
    int32_t f = INT32_MAX;
    for (int w = 0; w < THREADS / 64; ++w) {
      c += wcnt[w];
      f = min(f, wfirst[w]);
    }
    a.count[g] = c;
    /* the tile's first change point in the read, -1 if it has none */
    a.first_cp[g] = f == INT32_MAX ? -1 : (int32_t)(i0 + f);
  }
}

namespace {

/* exclusive scan of v over the workgroup (THREADS lanes); returns the prefix
 * and sets total */
__device__ __forceinline__ uint64_t block_exclusive_scan(uint64_t v, uint64_t *sh, uint64_t &total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint64_t inc = v;
  for (int d = 1; d < 64; d <<= 1) {
    const uint64_t o = __shfl_up(inc, d, 64);
    if (lane >= d) inc += o;
  }
  if (lane == 63) sh[wave] = inc;
  __syncthreads();
  uint64_t before = 0, all = 0;
  for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
    if (w < wave) before += sh[w];
    all += sh[w];
  }
  __syncthreads();
  total = all;
  return before + inc - v;
}

}  // namespace

/* One block scans all tiles and makes the reads' offsets too, four reads a thread at
 * most: 16 reads of 5 kb need 4 launches rather than 6, of 2 to 3 us each.  More reads
 * than tiles are empty reads, and one block is slow at many (200000: 1146 us a call
 * against 166 with a launch of their own). */
__host__ __device__ inline bool one_block_offsets(uint32_t blocks, int n_reads) {
  return blocks == 1 && n_reads <= SCAN_TILES;
}

/* first level: tiles [b*1024, (b+1)*1024), four consecutive per thread */
__global__ __launch_bounds__(THREADS) void k_ed_scan(DetectArgs a) {
  __shared__ uint64_t sh[THREADS / 64];
  const uint64_t t0 = (uint64_t)blockIdx.x * SCAN_TILES + 4u * threadIdx.x;
  /* (the plan lies in host memory: requested early) */
  const bool offsets = one_block_offsets(gridDim.x, a.n_reads);
  const uint32_t tf = offsets && (int)threadIdx.x <= a.n_reads ? a.tile_first[threadIdx.x] : 0;
  uint32_t c[4];
  uint64_t s = 0;
  for (int q = 0; q < 4; ++q) {
    c[q] = (t0 + q < a.n_tiles) ? a.count[t0 + q] : 0u;
    s += c[q];
  }
  uint64_t total;
  uint64_t p = block_exclusive_scan(s, sh, total);
  for (int q = 0; q < 4; ++q) {
    if (t0 + q < a.n_tiles) a.base[t0 + q] = p;
    p += c[q];
  }
  if (!offsets) {
    if (threadIdx.x == 0) a.block_sum[blockIdx.x] = total;
    return;
  }
  if (threadIdx.x == 0) {
    a.block_sum[0] = 0;
    a.block_sum[1] = total;
  }
  __syncthreads();
  for (int r = threadIdx.x; r <= a.n_reads; r += THREADS) {
    const uint32_t t = r == (int)threadIdx.x ? tf : a.tile_first[r];
    a.event_offset[r] = t < a.n_tiles ? a.base[t] : total;
  }
}

/* second level, one workgroup: exclusive scan of the block sums in place;
 * block_sum[n_blocks] receives the batch's event count */
__global__ __launch_bounds__(THREADS) void k_ed_scan_top(DetectArgs a, uint32_t n_blocks) {
  __shared__ uint64_t sh[THREADS / 64];
  uint64_t carry = 0;
  for (uint32_t b0 = 0; b0 < n_blocks; b0 += THREADS) {
    const uint32_t b = b0 + threadIdx.x;
    const uint64_t v = b < n_blocks ? a.block_sum[b] : 0;
    uint64_t total;
    const uint64_t p = block_exclusive_scan(v, sh, total);
    if (b < n_blocks) a.block_sum[b] = carry + p;
    carry += total;
  }
  if (threadIdx.x == 0) a.block_sum[n_blocks] = carry;
}

namespace {

/* a / b and the square root in double, rounded to nearest, for the operands that
 * arise here (without the general forms' care for tiny, huge and special ones).
 *
 * b: a whole number below 2^16, r its reciprocal to within an ulp or two.  The
 * residual a - q b is exact, and so is its share of the quotient to 2^-50 ulp,
 * while a / b lies at least 2^-17 ulp from the middle of two doubles, or on a
 * double. */
__device__ __forceinline__ double small_rcp(double b) {
  double r = __builtin_amdgcn_rcp(b); /* about 2^-23 */
  r = __builtin_fma(__builtin_fma(-b, r, 1.0), r, r);
  return __builtin_fma(__builtin_fma(-b, r, 1.0), r, r);
}
__device__ __forceinline__ double small_div(double a, double b, double r) {
  const double q = a * r;
  return __builtin_fma(__builtin_fma(-q, b, a), r, q);
}
/* v: 0, or a whole number below 2^64; Newton's iteration for v^-1/2, coupled with
 * that for v^1/2, and two corrections from the residual */
__device__ __forceinline__ double whole_sqrt(double v) {
  const double x = v == 0.0 ? 1.0 : v;
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  const double e = __builtin_fma(-h, g, 0.5);
  g = __builtin_fma(g, e, g);
  h = __builtin_fma(h, e, h);
  g = __builtin_fma(__builtin_fma(-g, g, x), h, g);
  g = __builtin_fma(__builtin_fma(-g, g, x), h, g);
  return v == 0.0 ? 0.0 : g;
}

}  // namespace

/* Events of a tile, a wavefront per tile, a lane 16 consecutive samples of it.
 *
 * What bounds it: the instructions per event (double precision) and per sample,
 * with the stores (12 B per event) behind them.  A workgroup per tile that stages
 * prefix sums of all samples in LDS, between barriers, and takes each event's two
 * divisions and root in their general forms needs 1050 us for 4000 reads of 5 kb
 * (284908 tiles); this form 334 us, 3.6 TB/s of samples and events.  Here a lane's prefix sums stay in registers, one wavefront
 * scan joins them, and only those at the tile's event starts go to LDS, in order,
 * for the lanes that take an event each; a wavefront waits for no other.
 *
 * MAXE: the most events that can start in a tile (peaks of a window w lie w or
 * more apart, so at most ceil(TS / w) of each detector, and the read's start). */
template <int MAXE, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void k_ed_events(DetectArgs a) {
  __shared__ uint4 lists[WAVES][MAXE + 1]; /* event starts: position, sums of x and x^2 before it */
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t g = blockIdx.x * WAVES + wave;
  if (g >= a.n_tiles) return;
  uint4 *list = lists[wave];
  const EdTile tl = a.tiles[g];
  const int64_t i0 = tl.i0;
  const int left = (int)((int64_t)tl.n - i0); /* samples from the tile's first to the read's end */
  const TileView tv = tile_view(a.raw + tl.s0, i0, tl.n);

  /* loads first: the first change points of the read's next 64 tiles, the flags
   * of the lane's boundaries, its samples, and 64 after the tile */
  const int f = (int64_t)g + 1 + lane < (int64_t)tl.g_end ? a.first_cp[g + 1 + lane] : -1;
  uint32_t bits = reinterpret_cast<const uint16_t *>(a.flags + (uint64_t)g * WORDS)[lane];
  int x[BPL];
  if (tv.hi > TS && (tv.lo < 0 || !tv.odd)) {
    uint32_t d[BPL / 2];
    word_pairs(tv, BPL * lane, d);
#pragma unroll
    for (int k = 0; k < BPL; ++k) x[k] = (k & 1) ? (int)d[k / 2] >> 16 : (int)(int16_t)d[k / 2];
  } else {
#pragma unroll
    for (int k = 0; k < BPL; ++k) x[k] = BPL * lane + k < left ? sample_at(tv, BPL * lane + k) : 0;
  }
  const int xt = TS + lane < left ? sample_at(tv, TS + lane) : 0;
  const uint64_t gbase = a.base[g] + a.block_sum[g / SCAN_TILES];

  /* no event starts in the tile: what runs through it is summed where it starts
   * (without this, tiles inside an event each summed the rest of it) */
  if (i0 == 0 && lane == 0) bits |= 1u; /* a read's first event starts at sample 0 */
  if (__ballot(bits != 0) == 0) return;

  /* the event that runs past the tile ends at the read's next change point: the
   * first change point of the first later tile that has one, or the read's end */
  int64_t end = left;
  uint64_t has = __ballot(f >= 0);
  if (has) {
    end = (int64_t)__builtin_amdgcn_readlane(f, __builtin_ctzll(has)) - i0;
  } else {
    for (int64_t h0 = (int64_t)g + 65; h0 < (int64_t)tl.g_end; h0 += 64) {
      const int fh = h0 + lane < (int64_t)tl.g_end ? a.first_cp[h0 + lane] : -1;
      has = __ballot(fh >= 0);
      if (has) {
        end = (int64_t)__builtin_amdgcn_readlane(fh, __builtin_ctzll(has)) - i0;
        break;
      }
    }
  }
  /* the sums of the samples past the tile up to there */
  int64_t ts, tq;
  if (end <= TS + 64) {
    const int v = TS + lane < end ? xt : 0;
    ts = __builtin_amdgcn_readlane(wave_scan(v), 63);
    tq = last_lane(wave_scan((long long)(v * v)));
  } else {
    long long s = xt, q = xt * xt;
    /* eight loads in flight: one wavefront is alone with a long event */
    int64_t k = TS + 64 + lane;
    for (; k + 7 * 64 < end; k += 8 * 64) {
      int v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = tv.x[k + 64 * u];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        s += v[u];
        q += v[u] * v[u];
      }
    }
    for (; k < end; k += 64) {
      const int v = tv.x[k];
      s += v;
      q += v * v;
    }
    ts = last_lane(wave_scan(s));
    tq = last_lane(wave_scan(q));
  }

  /* sums before each sample of the lane, then before the lane */
  int sp[BPL], s = 0;
  long long qp[BPL], q = 0;
#pragma unroll
  for (int k = 0; k < BPL; ++k) {
    sp[k] = s;
    qp[k] = q;
    s += x[k];
    q += x[k] * x[k];
  }
  const int si = wave_scan(s);
  const long long qi = wave_scan(q);
  const int ni = wave_scan((int)__popc(bits));
  const int n_ev = __builtin_amdgcn_readlane(ni, 63);
  uint4 *at = list + (ni - (int)__popc(bits));
#pragma unroll
  for (int k = 0; k < BPL; ++k) {
    if ((bits >> k) & 1u) {
      const long long qk = qi - q + qp[k];
      *at++ = make_uint4((uint32_t)(BPL * lane + k), (uint32_t)(si - s + sp[k]), (uint32_t)qk, (uint32_t)(qk >> 32));
    }
  }
  if (lane == 63) {
    const long long qk = qi + tq;
    list[n_ev] = make_uint4((uint32_t)end, (uint32_t)si + (uint32_t)ts, (uint32_t)qk, (uint32_t)((uint64_t)qk >> 32));
  }
  wave_exchange();

  const double off = (double)a.offset[tl.read];
  const double sc = (double)a.pa_scale[tl.read];
  for (int e = lane; e < n_ev; e += 64) {
    const uint64_t idx = gbase + (uint64_t)e;
    const uint4 e0 = list[e], e1 = list[e + 1];
    const int32_t len = (int32_t)(e1.x - e0.x);
    const int32_t s32 = (int32_t)(e1.y - e0.y);
    const int64_t qe = (int64_t)((((uint64_t)e1.w << 32) | e1.z) - (((uint64_t)e0.w << 32) | e0.z));
    const double dlen = (double)len;
    /* len^2 times the population variance, exact, rounded once to double:
     * below 2^16 samples S fits 32 bits and len * Q and S^2 stay below 2^62
     * (samples are 16-bit), so 64 bits hold it; longer events take 128 */
    double m, sd;
    if (len < 65536) {
      const double r = small_rcp(dlen);
      m = small_div((double)s32, dlen, r);
      sd = small_div(whole_sqrt((double)(uint64_t)((int64_t)len * qe - (int64_t)s32 * s32)), dlen, r);
    } else { /* the tile's last event: what of its sum lies in the tile, and past it */
      const int64_t se = (int64_t)(int32_t)(e1.y - (uint32_t)ts - e0.y) + ts;
      m = (double)se / dlen;
      const unsigned __int128 vv = (unsigned __int128)((__int128)len * qe - (__int128)se * se);
      const uint64_t hi = (uint64_t)(vv >> 64);
      double vd;
      if (hi == 0) {
        vd = (double)(uint64_t)vv;
      } else {
        /* keep the top 64 bits and a sticky bit: one rounding to double */
        const int k = 64 - __builtin_clzll(hi);
        const unsigned __int128 low = vv & ((((unsigned __int128)1) << k) - 1);
        const uint64_t top = (uint64_t)(vv >> k) | (low != 0 ? 1u : 0u);
        vd = __builtin_ldexp((double)top, k);
      }
      sd = __builtin_sqrt(vd) / dlen;
    }
    if (idx >= a.capacity) continue;
    float *ev = a.events + 3 * idx;
    ev[0] = (float)((m + off) * sc);
    ev[1] = (float)(sd * sc);
    ev[2] = (float)len;
  }
}

__global__ void k_ed_offsets(DetectArgs a, uint32_t n_blocks) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r > a.n_reads) return;
  const uint32_t t = a.tile_first[r];
  a.event_offset[r] = t < a.n_tiles ? a.base[t] + a.block_sum[t / SCAN_TILES] : a.block_sum[n_blocks];
}

uint32_t ed_scan_blocks(uint32_t n_tiles) { return (n_tiles + SCAN_TILES - 1) / SCAN_TILES; }

hipError_t launch_detect(const DetectArgs &a, hipStream_t st, hipEvent_t *tev) {
  const uint32_t nb = ed_scan_blocks(a.n_tiles);
  hipEvent_t e0 = tev ? tev[0] : nullptr, e1 = tev ? tev[1] : nullptr;
  hipEvent_t e2 = tev ? tev[2] : nullptr, e3 = tev ? tev[3] : nullptr;
  if (tev) {
    const hipError_t e = hipEventRecord(tev[4], st);
    if (e != hipSuccess) return e;
  }
  if (a.n_tiles > 0) {
    hipLaunchKernelGGL(k_ed_tiles, dim3((a.n_reads + 3) / 4), dim3(256), 0, st, a);
    /* the two streaming kernels take their start and end from their own
     * dispatch when timed */
    if (a.w_short == 3 && a.w_long == 8)
      hipExtLaunchKernelGGL(k_ed_detect, dim3((a.n_tiles + 3) / 4), dim3(THREADS), 0, st, e0, e1, 0, a);
    else
      hipExtLaunchKernelGGL(k_ed_detect_any, dim3(a.n_tiles), dim3(THREADS), 0, st, e0, e1, 0, a);
    hipLaunchKernelGGL(k_ed_scan, dim3(nb), dim3(THREADS), 0, st, a);
  } else if (tev) {
    (void)hipEventRecord(e0, st);
    (void)hipEventRecord(e1, st);
  }
  if (!one_block_offsets(nb, a.n_reads)) hipLaunchKernelGGL(k_ed_scan_top, dim3(1), dim3(THREADS), 0, st, a, nb);
  if (a.n_tiles > 0) {
    /* the event lists' room decides how many wavefronts a CU holds */
    const int most = (TS + a.w_short - 1) / a.w_short + (TS + a.w_long - 1) / a.w_long + 1;
    if (most <= 480)
      hipExtLaunchKernelGGL((k_ed_events<480, 4>), dim3((a.n_tiles + 3) / 4), dim3(256), 0, st, e2, e3, 0, a);
    else
      hipExtLaunchKernelGGL((k_ed_events<TS + 1, 2>), dim3((a.n_tiles + 1) / 2), dim3(128), 0, st, e2, e3, 0, a);
  } else if (tev) {
    (void)hipEventRecord(e2, st);
    (void)hipEventRecord(e3, st);
  }
  const int nr = a.n_reads + 1;
  if (!one_block_offsets(nb, a.n_reads)) hipLaunchKernelGGL(k_ed_offsets, dim3((nr + 255) / 256), dim3(256), 0, st, a, nb);
  if (tev) {
    const hipError_t e = hipEventRecord(tev[5], st);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

}  // namespace abea
