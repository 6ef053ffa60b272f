/*
 * abea_kernels.hip -- gfx950 kernels of Adaptive Banded Event Alignment.
 *
 * The thesis (Ch. 5 "GPU Accelerated Adaptive Banded Event Alignment")
 * splits the work into a pre-kernel (§5.4.1.1, Alg. 5.5: first bands and the
 * per-read "kcache" of model entries), a core-kernel (§5.4.1.2, Alg. 5.6-5.8:
 * the band loop, one thread block per read, four block barriers per band) and
 * a post-kernel (§5.4.1.3: one thread per read backtracks).  The same three
 * stages are here, re-designed for CDNA4:
 *
 *  k_prep      one workgroup per read: the read's status and, only where the
 *              band fill cannot read them in place (inputs at addresses of
 *              their own, e.g. mapped host memory, or events scaled to the
 *              model), a copy of the ranks and the event means.  The
 *              scaled model level of every k-mer position, mu' = fma(mean,
 *              scale, shift) (paragraph after Alg. 5.3), and its emission
 *              terms (the kcache) are made by the band fill itself, from
 *              the rank and the model entry it gathers.
 *  k_band      one 64-lane wavefront per read, no barrier and no score in
 *              memory.  K-mer k of a band lives in slot k mod N (N = 64*CPL >
 *              W; slot s is lane s / CPL, register s % CPL), so a cell's up
 *              neighbour is the same slot of the previous band and its left
 *              and diagonal neighbours are slot s-1 of the two previous bands:
 *              one DPP wave_ror:1 per band (the diagonal reuses the previous
 *              band's).  The slots keep their k-mers and are relabelled every
 *              few bands from a per-wave LDS k-mer ring; each band reads its
 *              events from an LDS event ring.  The band move (Suzuki-Kasahara
 *              rule) is a wave-uniform scalar decision.  Slots outside the band
 *              are cleared each band: every one of them to -inf, or (interior
 *              bands at two and four slots per lane, abea_interior.h) only the
 *              two beside the band.  Only two trace bits per slot reach HBM (two bit planes,
 *              32/CPL bands per 32-bit word).
 *  k_backtrack one wavefront per read walks the path, its trace cut into up to
 *              64 segments walked at once, one lane each, from guessed starts
 *              that are checked against the segment above; what differs is walked
 *              again, at once or one segment after the other.  The trace bits of
 *              cell (e, k) are in group (e+k)/G, lane (k mod N)/CPL.  The path is
 *              kept as two bits per band.
 *  k_align     the fused form: each wavefront fills a read's bands and then
 *              walks it, one read per wavefront or a persistent pool taking
 *              reads from a device work queue.
 *  k_scan/k_expand turn per-read path lengths into the caller's pair offsets
 *              and the path bits into its pairs.
 *
 * Arithmetic of a cell follows Alg. 5.2 and 5.3 exactly as the CPU reference
 * does: FP32, no contraction (-ffp-contract=off and the pragma below), the
 * emission as c - ((x - mu')^2 * h), the moves as (pred + lp) + em, and the
 * first maximum in the order diagonal, up, left.
 */
#include "abea_internal.h"
#include "abea_interior.h"

#include <hip/hip_ext.h>

#include <algorithm>
#include <climits>
#include <mutex>
#include <type_traits>

#pragma clang fp contract(off)

namespace abea {

#define ABEA_NINF (-__builtin_inff())

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <int CPL>
struct Log2 {
  static constexpr int v = CPL == 1 ? 0 : CPL == 2 ? 1 : CPL == 4 ? 2 : CPL == 8 ? 3 : 4;
};

/* lane l receives v of lane l-1, lane 0 receives lane 63 (DPP wave_ror:1).
 * Every lane has a source, so bound_ctrl changes nothing; it is set because
 * it lets the compiler fold the rotation into the instruction that uses it. */
__device__ __forceinline__ float rot_up(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x13C, 0xF, 0xF, true));
}
/* rot_up(l) + a and rot_up(d) + b, the rotations folded into the adds (two
 * v_add_f32_dpp, where a shared rotation would be a move and two adds).  The
 * s_nop gives the two wait states a DPP read needs after a VALU write of
 * its source, which the compiler does not track into inline assembly. */
__device__ __forceinline__ void add_rot2(float l, float a, float d, float b, float &lo, float &dout) {
  asm("s_nop 1\n\t"
      "v_add_f32_dpp %0, %2, %3 wave_ror:1 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %1, %4, %5 wave_ror:1 row_mask:0xf bank_mask:0xf"
      : "=&v"(lo), "=&v"(dout)
      : "v"(l), "v"(a), "v"(d), "v"(b));
}
__device__ __forceinline__ float rlane(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
__device__ __forceinline__ uint32_t rlane_u(uint32_t v, int lane) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}
/* per lane: bit set in `mask`, made on the scalar unit, selects if_set, else
 * if_clear (one v_cndmask) */
__device__ __forceinline__ float sel(float if_clear, float if_set, uint64_t mask) {
  float r;
  asm("v_cndmask_b32_e64 %0, %1, %2, %3" : "=v"(r) : "v"(if_clear), "v"(if_set), "s"(mask));
  return r;
}
/* the same for a mask that a vector compare made: two wait states first, which
 * the compiler does not track into inline assembly */
__device__ __forceinline__ float sel_cmp(float if_clear, float if_set, uint64_t mask) {
  float r;
  asm("s_nop 1\n\tv_cndmask_b32_e64 %0, %1, %2, %3" : "=v"(r) : "v"(if_clear), "v"(if_set), "s"(mask));
  return r;
}
/* a wave-uniform value held in a VGPR (one v_mov_b32) */
__device__ __forceinline__ float to_vgpr(float s) {
  float r;
  asm("v_mov_b32 %0, %1" : "=v"(r) : "s"(s));
  return r;
}
/* per lane: the largest of a, b and c (one v_max3_f32, no canonicalisation) */
__device__ __forceinline__ float vmax3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
/* per lane: the two trace planes shifted left by one, bit 0 of td set where s == d,
 * of tu where s == u: two compares and two v_addc, with the two wait states
 * between a compare and the v_addc that reads its mask (the compiler, given the
 * expression, makes a v_cndmask and a shift of each v_addc) */
__device__ __forceinline__ void shift_in(uint32_t &td, uint32_t &tu, float s, float d, float u) {
  uint64_t m;
  asm("v_cmp_eq_f32_e64 %2, %3, %4\n\t"
      "v_cmp_eq_f32_e32 vcc, %3, %5\n\t"
      "s_nop 0\n\t"
      "v_addc_co_u32_e64 %0, %2, %0, %0, %2\n\t"
      "v_addc_co_u32_e32 %1, vcc, %1, %1, vcc"
      : "+v"(td), "+v"(tu), "=&s"(m)
      : "v"(s), "v"(d), "v"(u)
      : "vcc");
}
/* the same for two slots, whose compares fill the wait states */
__device__ __forceinline__ void shift_in(uint32_t &td, uint32_t &tu, float s0, float d0, float u0, float s1, float d1,
                                         float u1) {
  uint64_t m0, m1, m2;
  asm("v_cmp_eq_f32_e64 %2, %5, %6\n\t"
      "v_cmp_eq_f32_e64 %3, %5, %7\n\t"
      "v_cmp_eq_f32_e64 %4, %8, %9\n\t"
      "v_cmp_eq_f32_e32 vcc, %8, %10\n\t"
      "v_addc_co_u32_e64 %0, %2, %0, %0, %2\n\t"
      "v_addc_co_u32_e64 %1, %3, %1, %1, %3\n\t"
      "v_addc_co_u32_e64 %0, %4, %0, %0, %4\n\t"
      "v_addc_co_u32_e32 %1, vcc, %1, %1, vcc"
      : "+v"(td), "+v"(tu), "=&s"(m0), "=&s"(m1), "=&s"(m2)
      : "v"(s0), "v"(d0), "v"(u0), "v"(s1), "v"(d1), "v"(u1)
      : "vcc");
}
__device__ __forceinline__ uint64_t ballot(bool b) { return __builtin_amdgcn_ballot_w64(b); }
/* lane `lane` of the result is `val` (uniform), the others keep `old`
 * (v_writelane; the compiler places the lane index in M0) */
__device__ int writelane(int val, int lane, int old) __asm("llvm.amdgcn.writelane.i32");

#define ABEA_NINF_BITS ((int)0xff800000)

/* Value held by slot `slot` of a band, as a scalar. */
template <int CPL>
__device__ __forceinline__ float read_slot(const float (&v)[CPL], int slot) {
  const int ln = slot >> Log2<CPL>::v;
  const int r = slot & (CPL - 1);
  /* read every register, then pick the scalar: a per-lane select over the
   * registers would be turned into an indexed (memory) access */
  float t = rlane(v[0], ln);
#pragma unroll
  for (int c = 1; c < CPL; ++c) {
    const float u = rlane(v[c], ln);
    t = (r == c) ? u : t;
  }
  return t;
}

/* ------------------------------------------------------------------ prep */

__global__ __launch_bounds__(256) void k_prep(const ReadDesc *__restrict__ reads,
                                              const float *__restrict__ events, int events_stride,
                                              const uint32_t *__restrict__ ranks,
                                              const uint64_t *__restrict__ in_addr,
                                              const float *__restrict__ scale,
                                              const float *__restrict__ shift,
                                              int scale_events,
                                              float *__restrict__ xmean,
                                              uint32_t *__restrict__ krank,
                                              int32_t *__restrict__ rstat,
                                              uint32_t *__restrict__ queue) {
  /* the work-queue counter of the alignment kernel that follows */
  if (blockIdx.x == 0 && threadIdx.x == 0 && queue) *queue = 0u;
  const ReadDesc rd = reads[blockIdx.x];
  if (rd.n_e <= 0 || rd.n_k <= 0) {
    if (threadIdx.x == 0) rstat[blockIdx.x] = READ_EMPTY;
    return;
  }
  /* a rank outside the model is found by the band fill, which reads every
   * rank of the read */
  if (threadIdx.x == 0) rstat[blockIdx.x] = READ_OK;
  /* the read's events and ranks: in the batch arrays at its offsets (12-byte
   * events with the mean first, or the means alone), or (in_addr) at
   * addresses of its own, where only the event means are stored */
  const int ev_stride = in_addr ? 1 : events_stride;
  const float *ev =
      in_addr ? reinterpret_cast<const float *>(in_addr[2 * rd.orig]) : events + (uint64_t)ev_stride * rd.ev_off;
  const uint32_t *rk =
      in_addr ? reinterpret_cast<const uint32_t *>(in_addr[2 * rd.orig + 1]) : ranks + rd.km_off;
  if (krank)
    for (int k = threadIdx.x; k < rd.n_k; k += blockDim.x) krank[rd.km_off + k] = rk[k];
  if (!xmean) return;
  if (scale_events) {
    /* per-read scaling (paragraph after Alg. 5.3), the events to the model:
     * x' = (x - shift) / scale, float32 subtract, correctly rounded divide */
    const float sc = scale[rd.orig];
    const float sh = shift[rd.orig];
    for (int e = threadIdx.x; e < rd.n_e; e += blockDim.x) {
      const float d = ev[(int64_t)ev_stride * e] - sh;
      xmean[rd.ev_off + e] = d / sc;
    }
  } else {
    for (int e = threadIdx.x; e < rd.n_e; e += blockDim.x) xmean[rd.ev_off + e] = ev[(int64_t)ev_stride * e];
  }
}

/* The arguments of the alignment kernels (their only parameter), read again
 * from the kernel argument segment, and the lane index made again: the
 * compiler may keep neither, nor what it derives from them, in registers
 * across this point, so the band fill and the walk of a fused kernel each hold
 * only what they use. */
typedef const __attribute__((address_space(4))) AlignArgs KernArgs;
__device__ __forceinline__ KernArgs &kernel_args() {
  KernArgs *p = (KernArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *p;
}
/* planned read s (the plan does not change while a kernel runs: scalar loads) */
__device__ __forceinline__ ReadDesc read_desc(const ReadDesc *reads, int s) {
  typedef const __attribute__((address_space(4))) u32x4 Piece;
  const Piece *p = (const Piece *)(uint64_t)(reads + s);
  u32x4 v[sizeof(ReadDesc) / sizeof(u32x4)];
#pragma unroll
  for (int q = 0; q < (int)(sizeof(ReadDesc) / sizeof(u32x4)); ++q) v[q] = p[q];
  ReadDesc d;
  __builtin_memcpy(&d, v, sizeof d);
  return d;
}
__device__ __forceinline__ int fresh_lane() {
  int l = threadIdx.x & 63;
  asm volatile("" : "+v"(l));
  return l;
}

/* ------------------------------------------------------------------ band */

/* Band move of the Suzuki-Kasahara rule from the bits of the two end cells
 * of the previous band, as a wave mask: all ones (k-mer move) if lo < hi,
 * else 0 (event move); when both are -inf the band parity decides, a k-mer
 * move for odd bands.  For odd bands hi is first raised to at least -FLT_MAX
 * (`nfm` holds -FLT_MAX in every lane): then lo < hi holds exactly when lo is
 * -inf too (no finite lo is below -FLT_MAX), and every other outcome is
 * unchanged.  The compare runs on the VALU with all lanes active, so its lane
 * mask is all ones or all zeros and its low half is the result.  The s_nop
 * gives the two wait states from the v_readlane of the end cells, which the
 * compiler does not track into inline assembly. */
template <bool ODD>
__device__ __forceinline__ uint64_t sk_move_mask(int lo, int hi, float nfm) {
  float tv;
  uint64_t cm;
  if (ODD)
    asm volatile(
        "s_nop 1\n\t"
        "v_max_f32 %[tv], %[h], %[nfm]\n\t"
        "v_cmp_lt_f32_e64 %[cm], %[lo], %[tv]"
        : [tv] "=&v"(tv), [cm] "=s"(cm)
        : [lo] "s"(lo), [h] "s"(hi), [nfm] "v"(nfm));
  else
    asm volatile(
        "s_nop 1\n\t"
        "v_mov_b32 %[tv], %[h]\n\t"
        "v_cmp_lt_f32_e64 %[cm], %[lo], %[tv]"
        : [tv] "=&v"(tv), [cm] "=s"(cm)
        : [lo] "s"(lo), [h] "s"(hi));
  return cm;
}

/* The same decision with the last end cell left in its register: one compare
 * of lo against every lane's value of that register (raised to -FLT_MAX for
 * odd bands), whose bit for the end cell's lane is the answer.  No readlane
 * and no move of the last end cell into a VGPR. */
template <bool ODD>
__device__ __forceinline__ uint64_t sk_cmp_lane(int lo, float hv, float nfm) {
  float tv;
  uint64_t cm;
  if (ODD)
    asm volatile(
        "s_nop 1\n\t"
        "v_max_f32 %[tv], %[h], %[nfm]\n\t"
        "v_cmp_lt_f32_e64 %[cm], %[lo], %[tv]"
        : [tv] "=&v"(tv), [cm] "=s"(cm)
        : [lo] "s"(lo), [h] "v"(hv), [nfm] "v"(nfm));
  else
    asm volatile("s_nop 1\n\tv_cmp_lt_f32_e64 %[cm], %[lo], %[h]" : [cm] "=s"(cm) : [lo] "s"(lo), [h] "v"(hv));
  return cm;
}

/* The register of slot (.. % CPL == r) of every lane, as one VGPR. */
template <int CPL>
__device__ __forceinline__ float pick(const float (&v)[CPL], int r) {
  float t = v[0];
#pragma unroll
  for (int c = 1; c < CPL; ++c) t = sel(t, v[c], ballot(r == c));
  return t;
}

/* The register holding slot `slot` of a band at four slots per lane, as one
 * VGPR: the register is chosen by the slot's two low bits in two levels of
 * selects, whose wave masks are made on the SALU. */
__device__ __forceinline__ float end_cell_reg4(const float (&v)[4], int slot) {
  uint64_t m0, m1;
  asm("s_bitcmp1_b32 %2, 0\n\t"
      "s_cselect_b64 %0, -1, 0\n\t"
      "s_bitcmp1_b32 %2, 1\n\t"
      "s_cselect_b64 %1, -1, 0"
      : "=&s"(m0), "=s"(m1)
      : "s"(slot)
      : "scc");
  const float a = sel(v[0], v[1], m0);
  const float b = sel(v[2], v[3], m0);
  return sel(a, b, m1);
}
/* Bits of the value held by slot `slot` at four slots per lane, as a scalar. */
__device__ __forceinline__ int end_cell_bits4(const float (&v)[4], int slot) {
  return __builtin_amdgcn_readlane(__float_as_int(end_cell_reg4(v, slot)), slot >> 2);
}

/* byte address in LDS of a shared array */
template <typename T>
__device__ __forceinline__ uint32_t lds_address(T *p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) T *)p;
}

/* Sizes of the band fill for CPL slots per lane.
 *   N   slots of the wave (64*CPL >= W + 2)
 *   G   bands per trace word (32/CPL, even)
 *   RX  entries of the event ring: holds every event of the band window
 *       plus the next G, in quarters of 64, one quarter spare (W + G <= RX - 128)
 *   RK  entries of the k-mer ring: holds k-mers K .. K+N+G, same rule
 *   S   sub-rings of the event ring: event e is in sub-ring e mod S.  At four
 *       slots per lane a register's slots hold k-mers of one residue mod 4,
 *       consecutive lanes k-mers 4 apart, so in a band the lanes of a
 *       register read events 4 apart: from one sub-ring, consecutive words
 *       (no LDS bank conflict), where a single ring would put them 4 words
 *       apart.  At two slots per lane the 2-way conflict of a single ring
 *       costs less than the sub-ring index arithmetic (measured on the
 *       W = 100 workloads); at one, lanes already read consecutive events.
 *   XS  floats of a sub-ring: RX/S entries and a mirror of its first G/S */
template <int CPL>
struct Geom {
  static constexpr int N = 64 * CPL;
  static constexpr int LC = Log2<CPL>::v;
  static constexpr int G = 32 / CPL;
  static constexpr int RX = CPL == 1 ? 256 : (128 * CPL > 1024 ? 1024 : 128 * CPL);
  static constexpr int RK = CPL == 1 ? 256 : 128 * CPL;
  static constexpr int S = CPL == 4 ? 4 : 1;
  static constexpr int LS = Log2<S>::v;
  static constexpr int XS = RX / S + G / S;
};

/* The walk.
 *   NP      16-byte pieces of a trace group (two lanes' words) kept per segment: the
 *           walk enters a group at a k-mer no higher than where it entered the
 *           group above, when the pieces were requested, and falls 2-3 k-mers per 8
 *           bands; a step outside them reads memory
 *   AHEAD   groups requested ahead when one segment is walked at a time
 *   SERIAL  trace groups up to which a path is walked in that way from the start:
 *           1024 bands, where 64 reads of 840 bands take 31 us at W = 100 for 40 in
 *           segments, and 6000 of 1680 bands 189 us for 94; at eight slots and more,
 *           with two or four bands a group, 2048 (6000 of 1680: 453 us for 604) */
template <int CPL>
struct WalkGeom {
  static constexpr int NP = CPL == 1 ? 8 : CPL == 2 ? 6 : CPL == 4 ? 3 : 2;
  static constexpr int AHEAD = 8;
  static constexpr int SERIAL = (CPL <= 4 ? 1024 : 2048) * CPL / 32;
};

/* LDS of one wavefront: the band fill's event ring (S sub-rings, each with a
 * mirror of its first G/S entries behind its end, so that a run of G reads
 * never wraps) and k-mer ring, or the walk's pieces of trace groups, one row
 * of 64 segments per piece; the two phases of a read never overlap. */
template <int CPL>
struct WaveLds {
  union {
    struct {
      float lx[Geom<CPL>::S * Geom<CPL>::XS];
      float4 lk[Geom<CPL>::RK];
    } band;
    u32x4 win[WalkGeom<CPL>::NP * 64];
  };
};

/* Band fill of one read whose status is READ_OK (Alg. 5.1 loop, Alg. 5.2,
 * 5.3), by the calling wavefront: writes the read's trace tiles, its
 * log-likelihood and cell count, and returns READ_OK or READ_BAND_LOST.
 *
 * Slot s (lane s / CPL, register s % CPL) holds k-mer kv(s) = K_r + ((s -
 * K_r) mod N), fixed from one refill to the next (every RF bands, RF <= N - W
 * and RF <= G): a k-mer that leaves the band keeps its slot until
 * the next refill relabels the slot as the k-mer N higher, which cannot enter
 * the band before then.  At a refill the wavefront loads each slot's k-mer
 * parameters (mu', c, h) from the k-mer ring and the LDS address of its event
 * at the refill band; band b after it reads the event of the slot from that
 * address + b (the event of a cell (e, k) in band i is i - 2 - k).
 *
 * Every slot computes a score each band; the slots outside the band must read
 * as -inf wherever a later cell of the band takes them as a neighbour.  Bands
 * with cells outside the DP table clear every slot outside the cells of the band
 * in the table, and so do interior bands unless CLEAR_EDGES.  With CLEAR_EDGES
 * (two or four slots per lane) interior bands run in abea_interior.h and clear
 * only k-mers K - 1 and K + W: the cells of the next band read band i at
 * k-mers K' - 1 .. K' + W - 1 and band i - 1 at K' - 1 .. K' + W - 2, with K'
 * = K or K + 1, so no other slot outside a band is ever read by a cell in one,
 * and what those slots hold (scores of k-mers outside the band, or NaN from
 * stale ring entries) never reaches the band, its end cells or the trace bits
 * of its cells.
 *
 * The interior code is for finite scores: it has no alternation for a move
 * between two cells of -inf, and a slot that it cleared could give a NaN.  Where
 * every event and k-mer parameter is within bounds (WILD below) every cell of a
 * band that lies in the table is finite, so neither arises.  A read that brings
 * another value into the rings is given up (READ_AGAIN) and filled once more with
 * `general` set, in which no band is interior: the code for the table's edges
 * takes any value. */
constexpr int READ_AGAIN = -1;
template <int CPL, int RPG, int CLEAR, bool TRIM>
__device__ __forceinline__ int band_read(KernArgs &a, const ReadDesc &rd, uint2 *trace,
                                         float *__restrict__ lx, float4 *__restrict__ lk, int general, int &e_end) {
  /* CLEAR: slot clearing of interior bands: 0 the window; else the two edge
   * slots, 1 + W mod CPL (the interior code is written for each) */
  constexpr bool CLEAR_EDGES = CLEAR != 0;
  static_assert(!CLEAR_EDGES || CPL == 2 || CPL == 4, "edge clearing needs two or four slots per lane");
  static_assert(CPL != 4 || Geom<CPL>::XS == EVENT_SUBRING, "the interior code knows the sub-rings' length");
  constexpr int N = Geom<CPL>::N;
  constexpr int LC = Geom<CPL>::LC;
  constexpr int G = Geom<CPL>::G;
  constexpr int RX = Geom<CPL>::RX;
  constexpr int RK = Geom<CPL>::RK;
  constexpr int S = Geom<CPL>::S;
  constexpr int LS = Geom<CPL>::LS;
  constexpr int XS = Geom<CPL>::XS;
  constexpr int RXS = RX / S;
  /* bands between slot refills; interior bands of edge kernels refill RPG times
   * per group (every NB bands), the others at most twice */
  constexpr int NB = G / RPG;
  constexpr int RF = RPG > 2 ? G / 2 : NB;
  static_assert(S == 1 || (G % S == 0 && RF % S == 0),
                "refills at band offsets that are multiples of S keep each register's sub-ring fixed");
  static_assert(RF >= 2 && RF % 2 == 0, "refill interval must be an even band count");

  const int lane = fresh_lane();
  const int n_e = rd.n_e, n_k = rd.n_k;
  const int W = a.W;

  /* vector copies of the move constants: a SIMD starts two float adds,
   * subtracts or multiplies of different waves per four cycles, but one whose
   * operand is a scalar register holds it for all four (2.2 against 4.2 cycles
   * an add with four waves per SIMD); and only with a vector second operand can
   * a rotation fold into the add (v_add_f32_dpp) */
  const float lp_skip = to_vgpr(rd.lp_skip), lp_stay = to_vgpr(rd.lp_stay), lp_step = to_vgpr(rd.lp_step);
  /* the read's event means, in place (every xstride-th float) or staged */
  const int xs = a.xstride;
  const float *__restrict__ xm = a.xsrc + (uint64_t)xs * rd.ev_off;
  /* the read's ranks and the model they index; each k-mer's parameters are
   * made here (the kcache of the paragraph after Alg. 5.3): mu' =
   * fma(mean, scale, shift) with one rounding, or the unscaled mean when the
   * events are scaled to the model, and the entry's emission terms c, h */
  const uint32_t *__restrict__ rk = a.ranks + rd.km_off;
  const float4 *__restrict__ mdl = reinterpret_cast<const float4 *>(a.model);
  const uint32_t n_model = a.n_model;
  const bool scale_ev = a.scale_events != 0;
  const float ksc = a.scale[rd.orig];
  const float ksh = a.shift[rd.orig];
  /* what this lane met: bit 0 a rank outside the model; edge kernels, bit 1 an
   * event or a k-mer's parameters in the rings beyond the bounds below (a NaN passes
   * no comparison).  Within them an emission is below 2^91 and a score of fewer
   * than 2^31 bands below 2^122 */
  constexpr uint32_t BAD_RANK = 1, WILD = 2;
  constexpr float MAX_LEVEL = 0x1p24f, MAX_TERM = 0x1p40f;
  uint32_t met = 0;
  /* 1 unless this is one of the longest reads, which run at raised priority (made
   * here, or the compiler keeps it in a vector register) */
  int calm;
  asm("s_cmp_lt_i32 %1, %2\n\ts_cselect_b32 %0, 1, 0" : "=s"(calm) : "s"(n_e + n_k), "s"(a.urgent_len) : "scc");
  const int H = W / 2;
  const float NI = ABEA_NINF;
  const float NFM = __int_as_float((int)0xff7fffff); /* -FLT_MAX */

  /* an event's mean and a k-mer's rank (positions outside the read take its first or
   * last: their slots are outside the table, whatever they hold never reaches a cell
   * of it.  Every lane loads, with no branch around it: a load that might not be there
   * would have the compiler wait for those before and after it alike) */
  auto ldx = [&](int e) -> float { return xm[(int64_t)xs * min(max(e, 0), n_e - 1)]; };
  auto ldr = [&](int k) -> uint32_t { return rk[min(max(k, 0), n_k - 1)]; };
  /* its model entry, gathered (a rank outside the model is noted, and
   * entry 0 read in its place) */
  auto gather = [&](uint32_t r) -> float4 {
    const bool ok = r < n_model;
    met |= ok ? 0u : BAD_RANK;
    return mdl[ok ? r : 0u];
  };
  /* the slot parameters (mu', c, h) of a gathered entry */
  auto kparam = [&](float4 m) -> float4 {
    return make_float4(scale_ev ? m.x : __builtin_fmaf(m.x, ksc, ksh), m.y, m.z, 0.0f);
  };
  /* event e = 64q + lane: sub-ring e mod S (the lane's low bits), entry
   * floor(e / S) mod RX/S */
  auto put_x = [&](int q, float v) {
    if constexpr (CLEAR_EDGES) met |= __builtin_fabsf(v) <= MAX_LEVEL ? 0u : WILD;
    float *sub = lx + (lane & (S - 1)) * XS;
    const int idx = ((q * 64 + lane) >> LS) & (RXS - 1);
    sub[idx] = v;
    if (idx < G / S) sub[RXS + idx] = v;
  };
  auto put_k = [&](int q, float4 v) {
    if constexpr (CLEAR_EDGES)
      met |= (__builtin_fabsf(v.x) <= MAX_LEVEL) & (__builtin_fabsf(v.y) <= MAX_TERM) &
                     (__builtin_fabsf(v.z) <= MAX_TERM)
                 ? 0u
                 : WILD;
    lk[(q * 64 + lane) & (RK - 1)] = v;
  };

  /* Trim states (the trim paragraph after Alg. 5.3): a column at k-mer -1
   * whose cell (e, -1) is (e-1, -1) + lp_trim, every event before the read
   * left unaligned; it lies in a band only while the band's first k-mer is
   * -1 or less, i.e. in bands with cells outside the table.  The first
   * k-mer is entered from it diagonally only (its left neighbour is -inf).
   * The end: end_best over the bands of the last k-mer's cells, the best of
   * (e, n_k-1) and the previous best with event e trimmed (ties to fewer
   * trims); end_u the end cell's event. */
  constexpr bool trim = TRIM;
  const float lp_trim = a.lp_trim;
  float end_best = ABEA_NINF;
  int end_u = -1;

  /* Band 1 (initialise_first_two_bands): band 0 has lower-left (W/2-1,
   * -1-W/2) and holds only the virtual origin (-1,-1) with score 0; band 1 is
   * band 0 moved one k-mer and is all -inf (with trim: but for the trim cell
   * (0, -1) at offset W/2-1).  K is the first k-mer of the latest band, E the
   * event of its first cell. */
  int K = -H;
  int E = H - 1;
  /* bits of the end cells of the latest band, for the next band's move:
   * band 1's are -inf, unless the trim cell is its first (W = 2, 3) */
  int lo_c = (trim && H == 1) ? __float_as_int(lp_trim) : ABEA_NINF_BITS, hi_c = ABEA_NINF_BITS;
  /* edge kernels: the next band's first k-mer, and its rotated neighbours, moved.
   * (The position after the move is kept, not the move: where the two meet in a
   * loop the compiler put the move into a vector register.) */
  int K_n = -H;
  float lf_n = NI, dg_n = NI;
  float Spp[CPL], Sp[CPL], PM[CPL], PC[CPL], PH[CPL];
  int kvs[CPL]; /* kv(slot), the k-mer the slot holds */
  int xb[CPL]; /* ring index of the slot's event at band b = 0 of the group */
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    const int kv = K + ((lane * CPL + c - K) & (N - 1));
    Spp[c] = (kv == -1) ? 0.0f : NI;                   /* band 0: the origin, k-mer -1 */
    Sp[c] = (trim && kv == -1) ? 0.0f + lp_trim : NI; /* band 1: the trim cell (0, -1) */
    PM[c] = PC[c] = PH[c] = 0.0f;
    kvs[c] = kv;
    xb[c] = 0;
  }

  if constexpr (CLEAR_EDGES) add_rot2(Sp[CPL - 1], lp_skip, Spp[CPL - 1], lp_step, lf_n, dg_n);

  /* Rings: event e in sub-ring e mod S at entry (e / S) mod (RX / S), k-mer
   * k at lk[k mod RK], written a quarter (64 entries) at a time; the quarter
   * after the top one waits in registers. */
  int xtop = (E + G) >> 6;
  int ktop = (K + N + G - 1) >> 6;
  /* (requested before the rings' first quarters, whose loads are waited for: with one
   * of these still in flight where the bands begin, the compiler has every later
   * refill wait for all loads and stores before it, 1% of a lone read) */
  float xpend = ldx((xtop + 1) * 64 + lane);
  /* the k-mer quarter after the top one: its model entries, gathered; the
   * one after that: its ranks (two loads in a chain, each a refill ahead) */
  float4 kpend = gather(ldr((ktop + 1) * 64 + lane));
  uint32_t rpend = ldr((ktop + 2) * 64 + lane);
  int q = (E - W + 1) >> 6;
  do {
    put_x(q, ldx(q * 64 + lane));
  } while (++q <= xtop);
  q = K >> 6;
  do {
    put_k(q, kparam(gather(ldr(q * 64 + lane))));
  } while (++q <= ktop);

  auto advance_rings = [&]() {
    if (((E + G) >> 6) > xtop) {
      ++xtop;
      put_x(xtop, xpend);
      xpend = ldx((xtop + 1) * 64 + lane);
    }
    if (((K + N + G - 1) >> 6) > ktop) {
      ++ktop;
      put_k(ktop, kparam(kpend));
      kpend = gather(rpend);
      rpend = ldr((ktop + 2) * 64 + lane);
    }
  };

  /* Relabel the slots for the current K (before band i's move) and load
   * their k-mer parameters and event addresses; b is the band's index in
   * its group, i = i0 + b. */
  auto refill = [&](int i, int b) {
    K = __builtin_amdgcn_readfirstlane(K);
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      const int d = (lane * CPL + c - K) & (N - 1);
      const int kv = K + d;
      kvs[c] = kv;
      const float4 p = lk[kv & (RK - 1)];
      PM[c] = p.x;
      PC[c] = p.y;
      PH[c] = p.z;
      /* the slot's event at this refill band i: e = i - 2 - kv, with e
       * mod S = (S - c) mod S for every lane (kv = c mod S, i = 2 mod S);
       * its sub-ring entry less the band offset (b is a multiple of S) */
      xb[c] = (((i - 2 - kv) >> LS) & (RXS - 1)) - (b >> LS);
    }
  };

  const int last = n_e + n_k;
  uint32_t TD = 0, TU = 0;
  float even_s = 0.0f, even_d = 0.0f, even_u = 0.0f; /* one slot per lane: an even band's, whose trace bits its odd one shifts in */
  uint64_t cells = 0;
  int edge_cells = 0; /* those of a group with cells outside the table */

  /* One band i = i0 + b: Spp = band i-2 (overwritten by band i), Sp = band
   * i-1.  INTERIOR: all W cells of band i are inside the DP table. */
  /* the events of the slots for band b (of the current refill interval) */
  auto load_x = [&](float(&x)[CPL], int b) {
    /* event e_ref + (b - b_ref) of slot register c: sub-ring (r0 + b) mod S,
     * entry xb[c] + (r0 + b) / S, with r0 = e_ref mod S = (S - c) mod S */
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      const int r0 = (S - (c & (S - 1))) & (S - 1);
      x[c] = lx[((r0 + b) & (S - 1)) * XS + xb[c] + ((r0 + b) >> LS)];
    }
  };

  /* fresh: the band opens a trace word (its first register's bits start the
   * words TD and TU; a full group's G*CPL bits fill them, so nothing carries
   * from one group to the next) */
  auto band = [&](auto interior_tag, float(&Spp)[CPL], const float(&Sp)[CPL], int i, int b,
                  const float(&X)[CPL], bool fresh) {
    constexpr bool INTERIOR = decltype(interior_tag)::value;
    static_assert(!(INTERIOR && CLEAR_EDGES), "edge kernels run interior bands in abea_interior.h");
    /* the band position is wave-uniform: keep it in SGPRs */
    K = __builtin_amdgcn_readfirstlane(K);
    /* Suzuki-Kasahara placement from the two end cells of band i-1 (taken
     * at the end of that band, into lo_c and hi_c); i0 is even, so i is odd
     * when b is.  The event of the first cell follows from K: e + k = i - 2
     * in band i. */
    const int lo = lo_c, hi = hi_c;
    if constexpr (CLEAR_EDGES) {
      K = K_n;
    } else {
      const uint64_t mv = (b & 1) ? sk_move_mask<true>(lo, hi, NFM) : sk_move_mask<false>(lo, hi, NFM);
      K -= __builtin_amdgcn_readfirstlane((int)(uint32_t)mv);
    }

    /* cells of band i inside the band and the table: k-mers kv with
     * wlo <= kv < wlo + wlen (one unsigned compare against the SGPR wlo) */
    int wlo = K, wlen = W;
    if constexpr (!INTERIOR) {
      wlo = max(K, max(0, i - 1 - n_e));
      wlen = max(0, min(K + W, min(n_k, i - 1)) - wlo);
      edge_cells += wlen;
    }
    /* slot s-1 of a register's first slot is the last register of lane l-1:
     * left (e, k-1) in band i-1 and diag (e-1, k-1) in band i-2, each with
     * its move's constant added */
    float lf0 = lf_n, dg0 = dg_n;
    if constexpr (!CLEAR_EDGES) add_rot2(Sp[CPL - 1], lp_skip, Spp[CPL - 1], lp_step, lf0, dg0);
    float nv[CPL]; /* band i; band i-2 is still read below */
    float sv[CPL]; /* band i before the window mask */
    float sd[CPL], su[CPL]; /* its candidates: diagonal and up */
    if (fresh) TD = TU = 0u;
    /* trim, in bands with cells outside the table: the first k-mer takes no
     * skip from the trim column (while the previous band may hold it), and
     * the trim cell (i-1, -1) of this band (while the band holds k-mer -1) */
    bool no_skip_in = false, trim_cell = false;
    if constexpr (!INTERIOR && TRIM) {
      no_skip_in = K <= 0;
      trim_cell = K <= -1 && i - 1 <= n_e - 1;
    }
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      const float x = X[c];
      const float up = Sp[c]; /* up (e-1, k): band i-1, slot s */
      /* left + lp_skip and diag + lp_step */
      const float lsk = (c == 0) ? lf0 : Sp[c - 1] + lp_skip;
      const float dst = (c == 0) ? dg0 : Spp[c - 1] + lp_step;
      /* Alg. 5.3 log-emission and Alg. 5.2 cell score */
      const float d = x - PM[c];
      const float t = d * d;
      const float u = t * PH[c];
      const float em = PC[c] - u;
      sd[c] = dst + em;
      su[c] = (up + lp_stay) + em;
      float sl = lsk;
      if constexpr (!INTERIOR && TRIM) {
        if (no_skip_in) sl = sel_cmp(sl, NI, ballot(kvs[c] == 0));
      }
      /* first maximum in the order D, U, L.  The value is the plain maximum
       * (scores are finite or -inf, never NaN or -0, so v_max3 gives the
       * bits of the first-maximum selects).  The trace bits say which
       * candidates equal it: D won iff sd is the maximum; otherwise U won iff
       * su is; otherwise L.  The compares stay off the chain from one band
       * to the next */
      sv[c] = vmax3(sd[c], su[c], sl);
      nv[c] = (uint32_t)(kvs[c] - wlo) < (uint32_t)wlen ? sv[c] : NI;
      if constexpr (!INTERIOR && TRIM) {
        if (trim_cell) nv[c] = sel_cmp(nv[c], up + lp_trim, ballot(kvs[c] == -1));
      }
      /* trace planes: the D bit, and the U bit (read only when D is clear) */
      if constexpr (CPL == 1) {
        if (b & 1) {
          shift_in(TD, TU, even_s, even_d, even_u, sv[c], sd[c], su[c]);
        } else {
          even_s = sv[c];
          even_d = sd[c];
          even_u = su[c];
        }
      } else if (c & 1)
        shift_in(TD, TU, sv[c - 1], sd[c - 1], su[c - 1], sv[c], sd[c], su[c]);
    }
    /* the end cells of this band for the next band's move.  Both lie in the
     * band; inside the table they are never masked, so they are read from
     * the unmasked scores, which keeps the window mask off the chain from
     * one band's move to the next */
    {
      const float(&src)[CPL] = INTERIOR ? sv : nv;
      const int sf = K & (N - 1);
      const int sh = (K + W - 1) & (N - 1);
      if constexpr (CLEAR_EDGES) {
        float r, h;
        if constexpr (CPL == 2) {
          const uint64_t m = (sf & 1) ? ~0ull : 0ull;
          r = sel(src[0], src[1], m);
          h = CLEAR == 2 ? r : sel(src[1], src[0], m); /* W odd: the same register's, else the other's */
        } else {
          r = end_cell_reg4(src, sf);
          h = end_cell_reg4(src, sh);
        }
        /* the next band is odd, and outside the table, if this one is even:
         * the last end cell raised to -FLT_MAX (see sk_move_mask) */
        const int lo1 = __builtin_amdgcn_readlane(__float_as_int(r), sf >> LC);
        const uint64_t cm = (b & 1) ? sk_cmp_lane<false>(lo1, h, NFM) : sk_cmp_lane<true>(lo1, h, NFM);
        K_n = K + __builtin_amdgcn_readfirstlane((int)(cm >> (sh >> LC)) & 1);
        add_rot2(nv[CPL - 1], lp_skip, Sp[CPL - 1], lp_step, lf_n, dg_n);
      } else if constexpr (CPL == 4) {
        lo_c = end_cell_bits4(src, sf);
        hi_c = end_cell_bits4(src, sh);
      } else {
        lo_c = __builtin_amdgcn_readlane(__float_as_int(pick<CPL>(src, sf & (CPL - 1))), sf >> LC);
        hi_c = __builtin_amdgcn_readlane(__float_as_int(pick<CPL>(src, sh & (CPL - 1))), sh >> LC);
      }
    }
    if constexpr (!INTERIOR && TRIM) {
      /* trim: band i holds (i-1-n_k, n_k-1) if it holds the last k-mer */
      if (i >= n_k + 1) {
        const float s_end =
            (n_k - 1 >= K && n_k - 1 <= K + W - 1) ? read_slot<CPL>(nv, (n_k - 1) & (N - 1)) : ABEA_NINF;
        const float t = end_best + lp_trim;
        if (t > s_end) {
          end_best = t;
        } else {
          end_best = s_end;
          end_u = i - 1 - n_k;
        }
      }
    }
#pragma unroll
    for (int c = 0; c < CPL; ++c) Spp[c] = nv[c];
  };

  /* A full group of G bands from band i: slot refill every RF bands; the
   * events of the next band pair are read from LDS while the current pair
   * computes (the scheduling barrier keeps the reads ahead).  Unrolled, so that the
   * instructions of a band fill the waits of the one before: a lone wavefront's band
   * at the table's edge takes 147 ns at W = 100 and 257 at W = 200, in a loop of one
   * pair 202 and 354. */
  auto group = [&](auto interior_tag, int i) {
    float xa[2][CPL], xn[2][CPL];
    refill(i, 0);
    load_x(xa[0], 0);
    load_x(xa[1], 1);
#pragma unroll
    for (int b = 0; b < G; b += 2) {
      const bool ahead = (b + 2 < G) && ((b + 2) % RF != 0);
      if (ahead) {
        load_x(xn[0], b + 2);
        load_x(xn[1], b + 3);
      }
      __builtin_amdgcn_sched_barrier(0);
      band(interior_tag, Spp, Sp, i + b, b, xa[0], b == 0);
      band(interior_tag, Sp, Spp, i + b + 1, b + 1, xa[1], false);
      if (b + 2 < G) {
        if ((b + 2) % RF == 0) {
          refill(i + b + 2, b + 2);
          load_x(xa[0], b + 2);
          load_x(xa[1], b + 3);
        } else {
#pragma unroll
          for (int c = 0; c < CPL; ++c) {
            xa[0][c] = xn[0][c];
            xa[1][c] = xn[1][c];
          }
        }
      }
    }
  };

  /* nb bands from band i, the first of a group: the last group of a read, which
   * may be a part.  Four at a time, the events of a pair of bands read while the
   * pair before computes. */
  auto few_bands = [&](int i, int nb) {
    static_assert(RF % 4 == 0 || RF == 2, "a refill interval ends at a quad or is a group");
    float xa[2][CPL], xc[2][CPL];
    TD = 0;
    TU = 0;
    refill(i, 0);
    load_x(xa[0], 0);
    load_x(xa[1], 1);
#pragma nounroll
    for (int b = 0;;) {
      load_x(xc[0], 2);
      load_x(xc[1], 3);
      band(std::false_type(), Spp, Sp, i + b, 0, xa[0], false);
      if (b + 1 == nb) break;
      band(std::false_type(), Sp, Spp, i + b + 1, 1, xa[1], false);
      if (b + 2 == nb) break;
      load_x(xa[0], 4);
      load_x(xa[1], 5);
      band(std::false_type(), Spp, Sp, i + b + 2, 0, xc[0], false);
      if (b + 3 == nb) break;
      band(std::false_type(), Sp, Spp, i + b + 3, 1, xc[1], false);
      b += 4;
      if (b == nb) break;
#pragma unroll
      for (int c = 0; c < CPL; ++c) xb[c] += 4 >> LS;
      if (b % RF == 0) {
        refill(i + b, 0);
        load_x(xa[0], 0);
        load_x(xa[1], 1);
      }
    }
    if (CPL == 1 && (nb & 1)) shift_in(TD, TU, even_s, even_d, even_u);
  };

  /* An interior group of an edge kernel: RPG refill intervals.  In each a lane's
   * slots hold CPL consecutive k-mers kv0 .. kv0+CPL-1 from a multiple of CPL: the
   * one K lies in, or a higher one (64*CPL - W - (CPL-1) >= NB keeps the k-mers
   * 64*CPL higher out of the band meanwhile).  kv0's parameters and the event of
   * the last of them at the interval's first band are all the lane needs. */
  auto interior_group = [&](int i) {
    if constexpr (CLEAR_EDGES) {
      Interior<CPL> v;
      v.stay = lp_stay;
      v.skip = lp_skip;
      v.step = lp_step;
      v.calm = calm;
      v.td = TD; /* a group's bits fill the words: nothing of these remains */
      v.tu = TU;
      v.lf = lf_n;
      v.dg = dg_n;
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        v.p[c] = Spp[c];
        v.q[c] = Sp[c];
      }
      const uint32_t bx = lds_address(lx), bk = lds_address(lk);
      auto interval = [&](auto res_tag, int ib) {
        constexpr int RES = decltype(res_tag)::value;
        const int kv0 = (K & -CPL) + ((lane * CPL - (K & -CPL)) & (N - 1));
        v.ak = bk + 16u * (uint32_t)(kv0 & (RK - 1));
        v.ax = bx + 4u * (uint32_t)(((ib - 2 - (kv0 + CPL - 1)) >> LS) & (RXS - 1));
        v.K = K_n;
        if constexpr (CPL == 2)
          interior<NB, CLEAR - 1>(v, W);
        else
          interior<NB, CLEAR - 1, RES>(v, W);
        K = __builtin_amdgcn_readfirstlane(v.K);
        K_n = K + v.mv;
      };
#pragma unroll
      for (int b = 0; b < G; b += NB) {
        if constexpr (CPL == 4 && NB == 2) {
          if (b & 2)
            interval(std::integral_constant<int, 3>(), i + b);
          else
            interval(std::integral_constant<int, 1>(), i + b);
        } else {
          interval(std::integral_constant<int, 1>(), i + b);
        }
      }
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        Spp[c] = v.p[c];
        Sp[c] = v.q[c];
      }
      TD = v.td;
      TU = v.tu;
      lf_n = v.lf;
      dg_n = v.dg;
    } else {
      group(std::true_type(), i);
    }
  };

  /* Groups of G bands (band i = 2 + t, group t / G): ring refill and interior
   * test once per group, one trace word per lane per group. */
  int i = 2;
  uint64_t g = 0;
  /* K at the start of each group, for the walk (every lane stores the same
   * word), in the read's path scratch, which the walk fills only after it has
   * read them */
  int *__restrict__ kpos = reinterpret_cast<int *>(a.scratch + rd.pr_off);
  /* interior bands clear CPL slots outside the band */
  const bool gap_ok = (N - W >= CPL) & (!CLEAR_EDGES | !general);
  while (i + G - 1 <= last) {
    K = __builtin_amdgcn_readfirstlane(K);
    E = i - 3 - K; /* band i - 1 is the latest */
    if constexpr (CLEAR_EDGES) {
      if (!general && ballot((met & WILD) != 0u)) return READ_AGAIN;
    }
    /* with trim the last k-mer stays out of interior bands, whose cells the
     * end recurrence does not read.  A group moves K and E up by G together, so
     * the next n groups are interior whatever their moves (256 at most: a wild
     * value ends the fill between two runs of them) */
    int n = 0;
    if (gap_ok & (K >= 0) & (E >= W - 1)) n = min(n_e - 1 - E, n_k - 1 - (int)trim - (K + W - 1)) / G;
    n = min(n, 256);
    if (n > 0) {
      cells += (uint64_t)W * (uint64_t)(G * n);
      do {
        E = i - 3 - K;
        advance_rings();
        kpos[g] = K;
        interior_group(i);
        trace[g * 64 + lane] = make_uint2(TD, TU);
        ++g;
        i += G;
      } while (--n > 0);
    } else {
      advance_rings();
      kpos[g] = K;
      group(std::false_type(), i);
      trace[g * 64 + lane] = make_uint2(TD, TU);
      cells += (uint32_t)edge_cells;
      edge_cells = 0;
      ++g;
      i += G;
    }
  }
  if (i <= last) {
    K = __builtin_amdgcn_readfirstlane(K);
    E = i - 3 - K;
    advance_rings();
    kpos[g] = K;
    const int nb = last - i + 1;
    few_bands(i, nb);
    cells += (uint32_t)edge_cells;
    const int sh = (G - nb) * CPL;
    trace[g * 64 + lane] = make_uint2(TD << sh, TU << sh);
  }
  if constexpr (CLEAR_EDGES) {
    if (!general && ballot((met & WILD) != 0u)) return READ_AGAIN;
  }

  /* terminal cell (n_e-1, n_k-1) is in the last band if its k-mer is; with
   * trim the end cell the end recurrence chose */
  float sc = ABEA_NINF;
  e_end = n_e - 1;
  if constexpr (TRIM) {
    sc = end_best;
    e_end = end_u;
  } else {
    float F[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) F[c] = (last & 1) ? Sp[c] : Spp[c];
    if (n_k - 1 >= K && n_k - 1 <= K + W - 1) sc = read_slot<CPL>(F, (n_k - 1) & (N - 1));
  }
  /* every rank of the read has passed through the k-mer ring: one outside
   * the model makes the read's outcome a bad rank, with no alignment */
  if (ballot((met & BAD_RANK) != 0u)) {
    if (lane == 0) {
      a.out_ll[rd.orig] = ABEA_NINF;
      if (a.out_cells) a.out_cells[rd.orig] = 0;
    }
    return READ_BAD_RANK;
  }
  if (lane == 0) {
    a.out_ll[rd.orig] = sc;
    if (a.out_cells) a.out_cells[rd.orig] = cells;
  }
  return (__float_as_int(sc) == ABEA_NINF_BITS) ? READ_BAND_LOST : READ_OK;
}

/* Outputs of a read whose band fill did not run (an empty read). */
__device__ __forceinline__ void band_skipped(KernArgs &a, const ReadDesc &rd) {
  if ((threadIdx.x & 63) == 0) {
    a.out_ll[rd.orig] = ABEA_NINF;
    if (a.out_cells) a.out_cells[rd.orig] = 0;
  }
}

/* Band fill alone, one wavefront per planned read. */
template <int CPL, int RPG, int EDGE, bool TRIM>
__global__ __launch_bounds__(64) void k_band(const AlignArgs a) {
  __shared__ WaveLds<CPL> lds;
  const int s = blockIdx.x;
  const ReadDesc rd = read_desc(a.reads, s);
  if (a.rstat[s] != READ_OK) {
    band_skipped(kernel_args(), rd);
    return;
  }
  /* the longest reads set the kernel's duration: let them issue first */
  const bool urgent = rd.n_e + rd.n_k >= a.urgent_len;
  if (urgent) __builtin_amdgcn_s_setprio(2);
  int st, e_end;
  for (int general = 0;; general = 1) {
    KernArgs &a1 = kernel_args();
    const ReadDesc r1 = read_desc(a1.reads, s);
    st = band_read<CPL, RPG, EDGE, TRIM>(a1, r1, a1.trace + r1.tr_off, lds.band.lx, lds.band.lk, general, e_end);
    if (__builtin_amdgcn_readfirstlane(st) != READ_AGAIN) break;
  }
  if (urgent) __builtin_amdgcn_s_setprio(0);
  if (threadIdx.x == 0) {
    a.rstat[s] = st;
    a.tend[s] = e_end;
  }
}

/* ------------------------------------------------------------- backtrack */

/* value of lane l+1 in lane l (the last lane keeps its own) */
__device__ __forceinline__ int from_above(int v) { return __shfl_down(v, 1, 64); }

/* Inclusive sum over the lanes of a wavefront. */
__device__ __forceinline__ uint32_t lane_scan(uint32_t v) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t o = __shfl_up(v, d, 64);
    if ((int)(threadIdx.x & 63) >= d) v += o;
  }
  return v;
}

/* The path's steps in one trace group, cell (t, k) first, its words in T (a lane's in
 * each lane): t and k on leaving it, and the path bits V and M of backtrack_read.
 * Each step is a run of up moves that ends with k's fall, on the scalar unit: the
 * words of k's lane, the run's length by one find-first-bit, 22 instructions and one
 * branch.  With TRIM the path may end here, at k = -1. */
template <int CPL, bool TRIM>
__device__ __forceinline__ void walk_group(uint2 T, int lower, int &t, int &k, uint32_t &V, uint32_t &M) {
  constexpr int LC = Log2<CPL>::v;
  uint32_t wd, wk, m, c;
  int b = t - lower + 1, pos, f; /* cells of the group's bands from t down */
  /* a run of n cells that ends at bit x of V.  s_bfm makes n bits, but none for 32 */
#define ABEA_WALK_RUN0(N, X) \
  "s_sub_u32 %[c], 32, " N "\n\ts_lshr_b32 %[c], -1, %[c]\n\ts_lshl_b32 %[c], %[c], " X "\n\t"
#define ABEA_WALK_RUN(N, X) "s_bfm_b32 %[c], " N ", " X "\n\t"
#define ABEA_WALK_POS0 "s_sub_u32 %[pos], 32, %[b]\n\t"
#define ABEA_WALK_POS(LC, CPL)                                                            \
  "s_and_b32 %[c], %[k], " #CPL "-1\n\ts_lshl" #LC "_add_u32 %[pos], %[b], %[c]\n\t"       \
  "s_sub_u32 %[pos], 31+" #CPL ", %[pos]\n\t"
#define ABEA_WALK(POS, RUN, LC, COL, END)                                                                 \
  asm(".Lstep_%=:\n\t"                                                                                     \
      "s_lshr_b32 %[c], %[k], " #LC "\n\t"                                                                 \
      "v_readlane_b32 %[wd], %[tx], %[c]\n\t"                                                              \
      "v_readlane_b32 %[wk], %[ty], %[c]\n\t" POS                                                          \
      "s_orn2_b32 %[wk], %[wd], %[wk]\n\t"                                                                 \
      "s_lshr_b32 %[m], %[wk], %[pos]\n\t"                                                                 \
      "s_and_b32 %[m], %[m], " #COL "\n\t"                                                                 \
      "s_cbranch_scc0 .Lup_%=\n\t"                                                                         \
      "s_ff1_i32_b32 %[f], %[m]\n\t"                                                                       \
      "s_add_u32 %[pos], %[pos], %[f]\n\t"                                                                 \
      "s_lshr_b32 %[f], %[f], " #LC "\n\t" /* the up moves */                                              \
      "s_add_u32 %[f], %[f], 1\n\t"                                                                        \
      "s_sub_u32 %[b], %[b], %[f]\n\t" RUN("%[f]", "%[b]")                                                 \
      "s_or_b32 %[V], %[V], %[c]\n\t"                                                                      \
      "s_bitset1_b32 %[M], %[b]\n\t"                                                                       \
      "s_sub_u32 %[k], %[k], 1\n\t"                                                                        \
      "s_bitcmp1_b32 %[wd], %[pos]\n\t"                                                                    \
      "s_subb_u32 %[b], %[b], 0\n\t" END                                                                   \
      "s_cmp_gt_i32 %[b], 0\n\t"                                                                           \
      "s_cbranch_scc1 .Lstep_%=\n\t"                                                                       \
      "s_branch .Lout_%=\n"                                                                                \
      ".Lup_%=:\n\t" /* up to the group's end */                                                           \
      "s_mov_b32 %[f], 0\n\t" RUN("%[b]", "%[f]")                                                          \
      "s_or_b32 %[V], %[V], %[c]\n\t"                                                                      \
      "s_mov_b32 %[b], 0\n"                                                                                \
      ".Lout_%=:\n"                                                                                        \
      : [k] "+&s"(k), [V] "+&s"(V), [M] "+&s"(M), [wd] "=&s"(wd), [wk] "=&s"(wk), [m] "=&s"(m), [c] "=&s"(c), \
        [b] "+&s"(b), [pos] "=&s"(pos), [f] "=&s"(f)                                                        \
      : [tx] "v"(T.x), [ty] "v"(T.y)                                                                        \
      : "scc")
#define ABEA_WALK_TRIM(POS, RUN, LC, COL)                                                                       \
  if constexpr (TRIM)                                                                                      \
    ABEA_WALK(POS, RUN, LC, COL, "s_cmp_lt_i32 %[k], 0\n\ts_cbranch_scc1 .Lout_%=\n\t");                       \
  else                                                                                                     \
    ABEA_WALK(POS, RUN, LC, COL, "")
  if constexpr (LC == 0) {
    ABEA_WALK_TRIM(ABEA_WALK_POS0, ABEA_WALK_RUN0, 0, 0xffffffff);
  } else if constexpr (LC == 1) {
    ABEA_WALK_TRIM(ABEA_WALK_POS(1, 2), ABEA_WALK_RUN, 1, 0x55555555);
  } else if constexpr (LC == 2) {
    ABEA_WALK_TRIM(ABEA_WALK_POS(2, 4), ABEA_WALK_RUN, 2, 0x11111111);
  } else if constexpr (LC == 3) {
    ABEA_WALK_TRIM(ABEA_WALK_POS(3, 8), ABEA_WALK_RUN, 3, 0x01010101);
  } else {
    ABEA_WALK_TRIM(ABEA_WALK_POS(4, 16), ABEA_WALK_RUN, 4, 0x00010001);
  }
  t = lower - 1 + b;
#undef ABEA_WALK_RUN0
#undef ABEA_WALK_RUN
#undef ABEA_WALK_POS0
#undef ABEA_WALK_POS
#undef ABEA_WALK
#undef ABEA_WALK_TRIM
}

/* Backtrack of one read (Alg. 5.1, after the band loop) by the calling
 * wavefront, from its trace tiles: writes the path as bits (path scratch), its
 * length, the trace groups it covers and the read's final status (and -inf as
 * log-likelihood if the walk fails).  The walk starts at (e_start, n_k-1):
 * (n_e-1, n_k-1), or with TRIM the end cell the band fill chose; it ends at the
 * origin, or with TRIM on reaching the trim column k = -1 (whose cells are not
 * pairs).
 *
 * What bounds it: a step needs the trace word of its cell, and the next cell
 * depends on it, so one walk is a chain of load, decode, move (60 ns a cell on the
 * scalar unit, a quarter of a long read's time).  Here the trace groups are cut into
 * up to 64 segments, one lane each, walked at once.  Where a segment's walk starts is
 * known only when the segment above is done, so each lane starts W bands higher
 * (WALK_OVERLAP at least), from the middle of the band there (the K the band fill
 * noted): the best paths to the cells of a band come from one cell a few dozen bands
 * below, so by the segment's top the guess has met the path.  That is checked, not
 * assumed: a segment is wrong whose walk entered it elsewhere than the segment above
 * left its own, the topmost being exact from the start.  The wrong ones are walked
 * again, all at once, while that helps: a lane that was right but for the one above it
 * is put right by it.  Where paths do not meet at all (events that fit every k-mer,
 * or none) it does not help, and what is wrong is walked one segment after the other
 * by the whole wavefront (walk_group), which also takes short paths from the start.
 * The path is then the one cell-by-cell walk's, whatever the guesses.
 *
 * At once: all lanes take a group at a time.  A step handles a run of up moves:
 * the run ends at the first cell of the column whose move lowers k (D bit, or
 * no U bit: wk = D | ~U), found by one find-first-bit over the column's bits of
 * the word.  The words a lane needs next lie in a few 16-byte pieces of the
 * group below, requested while the current group is walked (WalkGeom) and kept
 * in LDS; a group takes 0.9 us.  One segment at a time: the same steps, 50 ns each,
 * the groups' words requested AHEAD groups before.
 * Measured (walk kernel): one read of 8000 k-mers 66 us at W = 100 (one cell after
 * the other 888); 64 reads of 8000 k-mers whose events fit every k-mer 645 us (walked
 * again segment by segment at once 1286), of random events 560; 20000 reads of 112
 * bands 54 us (in segments 82); one of 60000 k-mers at W = 250 783 us (with
 * WALK_OVERLAP for every W 5640).
 *
 * Path scratch of a read: one word pair (V, M) per group, bit b for the cell of
 * band g*G + b: V set if the path visits the band, M if k falls on leaving that
 * cell; then, with more than one segment, the count of path cells and of M bits
 * below each segment. */
template <int CPL, bool TRIM>
__device__ __forceinline__ void backtrack_read(KernArgs &a, const ReadDesc &rd, int status, int e_start,
                                               const uint2 *tr, u32x4 *win) {
  constexpr int N = 64 * CPL;
  constexpr int LC = Log2<CPL>::v;
  constexpr int LG = 5 - LC;           /* log2(G) */
  constexpr int G = 1 << LG;           /* bands per trace group */
  typedef WalkGeom<CPL> WG;
  constexpr int NP = WG::NP;
  constexpr uint32_t COL = CPL == 1 ? 0xffffffffu : CPL == 2 ? 0x55555555u : CPL == 4 ? 0x11111111u
                         : CPL == 8 ? 0x01010101u : 0x00010001u; /* one slot's bits of a trace word */

  const int lane = fresh_lane();
  const int orig = rd.orig;
  if (status != READ_OK) {
    if (lane == 0) {
      a.path_len[orig] = 0;
      a.path_src[orig] = 0;
      a.out_status[orig] = status;
    }
    return;
  }
  const int OV = max(WALK_OVERLAP, a.W) >> LG; /* groups a lane starts above its segment */
  const int n_e = rd.n_e, n_k = rd.n_k;
  const int t_start = __builtin_amdgcn_readfirstlane(e_start) + n_k - 1;
  const int gtop = t_start >> LG; /* the path's last trace group */
  const int groups = (n_e + n_k - 1 + G - 1) >> LG;
  int sl; /* groups per segment */
  const int nseg = path_segments(gtop + 1, sl);
  int2 *pw = a.scratch + rd.pr_off;

  /* this lane's segment: groups glo .. ghi (lanes past the last segment have
   * none), and where its walk starts */
  const int glo = lane * sl;
  const int ghi = lane < nseg ? min(gtop, glo + sl - 1) : glo - 1;
  int g = ghi + OV;
  int t = t_start, k = n_k - 1;
  if (lane >= nseg) {
    g = glo - 1;
  } else if (g >= gtop) {
    g = gtop;
  } else {
    t = (g << LG) + G - 1;
    k = reinterpret_cast<const int *>(pw)[g + 1] + a.W / 2;
    k = max(max(0, t - n_e + 1), min(k, min(n_k - 1, t)));
  }
  if (lane < nseg) ++g;
  asm volatile("" ::: "memory"); /* the noted K are read before the path is written over them */

  uint32_t nv = 0, nm = 0;     /* path cells and M bits of the segment */
  int t_in = INT_MIN, k_in = 0; /* where the walk entered the segment */
  uint64_t wrong = 1ull << (nseg - 1); /* the segments to be walked from where the one above left its own */
  /* (the wrong segments are walked again at once while that leaves a quarter fewer) */
#pragma nounroll
  for (int before = nseg; gtop + 1 > WG::SERIAL;) {
    /* every lane from (t, k) in group g-1 down to the end of its segment.  The
     * pieces of a group around k-mer kk hold the words of lanes a0, a0-1, ...
     * with a0 odd, so that a piece's two words never straddle the ring's end;
     * the first pass only requests them */
    int a0 = 0;
    while (ballot(g >= glo)) {
      const bool on = g >= glo;
      const int lower = g << LG;
      if (g == ghi) {
        t_in = t;
        k_in = k;
      }
      const int a1 = ((k & (N - 1)) >> LC) | 1;
      /* (lanes that are done read some group of the read: no branch around
       * the loads, whose registers would double) */
      u32x4 pf[NP];
      const uint2 *row = tr + (uint64_t)min(max(g - 1, 0), gtop) * 64;
#pragma unroll
      for (int p = 0; p < NP; ++p) pf[p] = *reinterpret_cast<const u32x4 *>(row + ((a1 - 1 - 2 * p) & 63));
      uint32_t V = 0, M = 0;
      for (;;) {
        const bool act = on && t >= lower && !(TRIM && k < 0);
        if (!ballot(act)) break;
        if (act) {
          const int w = (k & (N - 1)) >> LC;
          const int rel = (a0 - w) & 63;
          uint2 T;
          if (rel < 2 * NP)
            T = reinterpret_cast<const uint2 *>(win)[((rel >> 1) * 64 + lane) * 2 + (w & 1)];
          else
            T = tr[(uint64_t)g * 64 + w];
          /* the cell of band lower + b, slot k: bit 31 - (b * CPL + k mod CPL) */
          const int b = t - lower;
          const int pos = 31 - ((b << LC) + (k & (CPL - 1)));
          const uint32_t m = ((T.x | ~T.y) >> pos) & COL;
          const int j = min((uint32_t)(__ffs(m) - 1) >> LC, (uint32_t)b + 1u); /* up moves */
          const bool found = j <= b; /* else the run leaves the group */
          const int bl = found ? b - j : 0;
          V |= ((2u << b) - 1u) & ~((1u << bl) - 1u);
          if (found) {
            M |= 1u << bl;
            t -= 1 + (int)((T.x >> (pos + (j << LC))) & 1u);
            k -= 1;
          }
          t -= j;
        }
      }
      if (on && g <= ghi) {
        nv += (uint32_t)__popc(V);
        nm += (uint32_t)__popc(M);
        pw[g] = make_int2((int)V, (int)M);
      }
#pragma unroll
      for (int p = 0; p < NP; ++p) win[p * 64 + lane] = pf[p];
      a0 = a1;
      if (on) --g;
    }
    /* a lane agrees with the one above if it entered its segment where that
     * one left its own */
    const int ta = from_above(t), ka = from_above(k);
    const bool off = lane < nseg - 1 && (t_in != ta || k_in != ka);
    wrong = ballot(off);
    const int count = __builtin_popcountll(wrong);
    if (count == 0 || 4 * count > 3 * before) break;
    before = count;
    if (off) {
      g = ghi + 1;
      t = ta;
      k = ka;
      nv = nm = 0;
    }
  }
  /* one cell after the other: the topmost wrong segment, then those below it until
   * the walk enters one where it was entered before; then the next wrong one */
  while (wrong) {
    constexpr int D = WG::AHEAD;
    int L = 63 - __builtin_clzll(wrong);
    int ts = t_start, ks = n_k - 1;
    if (L < nseg - 1) {
      ts = (int)rlane_u((uint32_t)t, L + 1);
      ks = (int)rlane_u((uint32_t)k, L + 1);
    }
    int gs = min(gtop, L * sl + sl - 1), gl = L * sl;
    uint2 T[D]; /* the words of groups gs, gs-1, .., one lane's in each lane */
    auto row = [&](int q) { return tr[(uint64_t)max(q, 0) * 64 + lane]; };
#pragma unroll
    for (int d = 0; d < D; ++d) T[d] = row(gs - d);
    uint32_t cv = 0, cm = 0;
    bool met = false;
    do {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        const int lower = gs << LG;
        uint32_t V = 0, M = 0;
        if (!(TRIM && ks < 0)) walk_group<CPL, TRIM>(T[d], lower, ts, ks, V, M);
        pw[gs] = make_int2((int)V, (int)M);
        cv += (uint32_t)__builtin_popcount(V);
        cm += (uint32_t)__builtin_popcount(M);
        T[d] = row(gs - D);
        if (TRIM && ks < 0) { /* the path's end: nothing below */
          for (int q = gs - 1 - lane; q >= 0; q -= 64) pw[q] = make_int2(0, 0);
          nv = lane == L ? cv : lane < L ? 0 : nv;
          nm = lane == L ? cm : lane < L ? 0 : nm;
          t = lane == 0 ? ts : t;
          k = lane == 0 ? ks : k;
          L = -1;
          met = true;
          break;
        }
        if (gs == gl) { /* the segment's end */
          if (lane == L) {
            t = ts;
            k = ks;
            nv = cv;
            nm = cm;
          }
          cv = cm = 0;
          --L;
          gl -= sl;
          met = L < 0 || ((int)rlane_u((uint32_t)t_in, L) == ts && (int)rlane_u((uint32_t)k_in, L) == ks);
          if (met) break;
        }
        --gs;
      }
    } while (!met);
    wrong &= L < 0 ? 0 : (1ull << L) - 1ull;
  }
  const int t_end = (int)rlane_u((uint32_t)t, 0), k_end = (int)rlane_u((uint32_t)k, 0);
  const bool ok = k_end == -1 && (TRIM ? t_end >= -2 : t_end == -2);
  /* path cells and M bits below each segment */
  const uint32_t sv = lane_scan(nv), sm = lane_scan(nm);
  if (nseg > 1 && lane < nseg) pw[groups + lane] = make_int2((int)(sv - nv), (int)(sm - nm));
  if (lane == 63) {
    a.path_len[orig] = ok ? (uint64_t)sv : 0;
    a.path_src[orig] = (uint64_t)(gtop + 1);
    a.out_status[orig] = ok ? READ_OK : READ_BAND_LOST;
    if (!ok) a.out_ll[orig] = ABEA_NINF;
  }
}

/* Backtrack alone, one wavefront per planned read. */
template <int CPL, bool TRIM>
__global__ __launch_bounds__(64) void k_backtrack(const AlignArgs a) {
  __shared__ WaveLds<CPL> lds;
  const int s = blockIdx.x;
  const ReadDesc rd = read_desc(a.reads, s);
  backtrack_read<CPL, TRIM>(kernel_args(), rd, a.rstat[s], TRIM ? a.tend[s] : rd.n_e - 1, a.trace + rd.tr_off, lds.win);
}

/* ----------------------------------------------------------------- fused */

/* Wavefronts per SIMD that the fused kernel's registers must leave room for
 * (the compiler would take more registers for the bands at the table's edges,
 * which are few).  At two and four slots per lane also the most it may leave room
 * for: where a launch brings five a SIMD (16 batches in flight in pools of 320), a
 * sixth place lets the wavefronts settle six on some SIMDs and four on others, whose
 * full ones end last (4000 reads a batch, W = 100: 2510 GCUPS with 78 registers and
 * six places, 2567 with five). */
constexpr int waves_per_simd(int cpl, bool trim) {
  return cpl == 1 ? (trim ? 4 : 5) : cpl == 2 ? 5 : cpl == 4 ? 4 : cpl == 8 ? 2 : 1;
}
constexpr int most_per_simd(int cpl, bool trim) { return cpl == 2 || cpl == 4 ? waves_per_simd(cpl, trim) : 8; }

/* Band fill and backtrack of a read by one wavefront, with a device work
 * queue.  Worker w (wavefront w of the grid, w < n_workers) first aligns
 * planned read w, then takes reads n_workers + q for q = 0, 1, ... from the
 * queue counter until they run out.  Reads are planned longest first, so
 * every later read fits the trace slab of the worker's first read: worker w
 * keeps read w's trace region for all its reads.  n_workers = n_reads is the
 * plain one-launch form; fewer workers bound the trace memory (admission by
 * traceback bytes) and let the longest reads of the batch overlap the rest. */
template <int CPL, int RPG, int WPG, int EDGE, bool TRIM>
__global__ __launch_bounds__(64 * WPG)
    __attribute__((amdgpu_waves_per_eu(waves_per_simd(CPL, TRIM), most_per_simd(CPL, TRIM)))) void k_align(
        const AlignArgs a) {
  __shared__ WaveLds<CPL> lds[WPG];
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int w = blockIdx.x * WPG + wv;
  if (w >= a.n_workers) return;
  int s = w, general = 0;
  for (;;) {
    KernArgs &a1 = kernel_args();
    if (s >= a1.n_reads) break;
    int st = a1.rstat[s];
    int e_end;
    {
      const ReadDesc rd = read_desc(a1.reads, s);
      /* the longest reads set the kernel's duration: let them issue first */
      if (rd.n_e + rd.n_k >= a1.urgent_len) __builtin_amdgcn_s_setprio(2);
      e_end = rd.n_e - 1;
      if (st == READ_OK)
        st = band_read<CPL, RPG, EDGE, TRIM>(a1, rd, a1.trace + read_desc(a1.reads, w).tr_off, lds[wv].band.lx,
                                             lds[wv].band.lk, general, e_end);
      else
        band_skipped(a1, rd);
    }
    if constexpr (EDGE != 0) {
      general = __builtin_amdgcn_readfirstlane(st) == READ_AGAIN;
      if (general) continue;
    }
    /* the walk reads back what this wavefront's lanes just stored; keep the
     * compiler from moving loads above the stores */
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
    KernArgs &a2 = kernel_args();
    backtrack_read<CPL, TRIM>(a2, read_desc(a2.reads, s), st, e_end, a2.trace + read_desc(a2.reads, w).tr_off,
                              lds[wv].win);
    __builtin_amdgcn_s_setprio(0);
    asm volatile("" ::: "memory");
    uint32_t q = 0;
    if ((threadIdx.x & 63) == 0) q = atomicAdd(a2.queue, 1u);
    s = a2.n_workers + (int)__builtin_amdgcn_readfirstlane(q);
  }
}

/* -------------------------------------------------------- scan + expand */

/* Both kernels run as single-wavefront workgroups: while other batches'
 * alignment waves hold the chip, a one-wave group takes the first free wave
 * slot, where a multi-wave group would wait for a CU with that many free
 * slots at once. */

/* Exclusive scan of n lengths, and their total.  The wavefront takes 512 at a
 * time, 8 consecutive per lane, with the next 512 requested: a lane that walks
 * its own n / 64 lengths one by one waits for each load (20000 reads: 170 us,
 * this 43). */
__global__ __launch_bounds__(64) void k_scan(const uint64_t *__restrict__ len, int n,
                                             uint64_t *__restrict__ off) {
  constexpr int U = 8;
  const int lane = threadIdx.x;
  uint64_t v[U], nx[U];
#pragma unroll
  for (int u = 0; u < U; ++u) nx[u] = lane * U + u < n ? len[lane * U + u] : 0;
  uint64_t carry = 0;
  for (int b = 0; b < n; b += 64 * U) {
    const int r = b + lane * U;
    uint64_t sum = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      v[u] = nx[u];
      sum += v[u];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) nx[u] = r + 64 * U + u < n ? len[r + 64 * U + u] : 0;
    uint64_t inc = sum; /* inclusive scan of the 64 lane sums */
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint64_t w = __shfl_up(inc, d, 64);
      if (lane >= d) inc += w;
    }
    uint64_t run = carry + inc - sum;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (r + u < n) off[r + u] = run;
      run += v[u];
    }
    carry += __shfl(inc, 63, 64);
  }
  if (lane == 63) off[n] = carry;
}

/* A read's pairs from its path bits (see backtrack_read), into its place in
 * the caller's array.  The cell of a visited band t has k = -1 + (M bits of the
 * path up to and with it) and e = t - k.  gridDim.y wavefronts per planned
 * read (launch_expand), each taking a run of whole segments, so that the longest
 * reads do not leave one wavefront writing megabytes at the end of the kernel.
 * A wavefront takes up to 64 groups at a time (1024 bands), one per lane: the
 * groups' counts are scanned over the lanes, each lane makes its cells into LDS, and
 * the wavefront stores them coalesced.  Bound by the 8 bytes per pair written: the
 * 1.2 G cells of a 20000-read job (0.5 to 200 kb) in 2.9 ms (3.4 TB/s), where
 * copying pairs from a scratch took 3.9 ms. */
constexpr int EXPAND_BANDS = 1024;
__global__ __launch_bounds__(64) void k_expand(const ReadDesc *__restrict__ reads, const int2 *__restrict__ scratch,
                                               const uint64_t *__restrict__ src,
                                               const uint64_t *__restrict__ off, int lg,
                                               int2 *__restrict__ pairs) {
  __shared__ int2 cell[EXPAND_BANDS];
  const ReadDesc rd = reads[blockIdx.x];
  const int lane = threadIdx.x;
  uint64_t o = off[rd.orig];
  if (off[rd.orig + 1] == o) return; /* no path */
  const int ng = (int)src[rd.orig];
  int sl;
  const int nseg = path_segments(ng, sl);
  const int per = (nseg + (int)gridDim.y - 1) / (int)gridDim.y; /* segments per wavefront */
  const int s0 = (int)blockIdx.y * per;
  if (s0 >= nseg) return;
  const int g1 = min(ng, (s0 + per) * sl);
  const int2 *pw = scratch + rd.pr_off;
  int2 *__restrict__ out = pairs + o;
  uint32_t idx = 0; /* path cells before the chunk */
  int k = -1;       /* k after them */
  if (nseg > 1) {
    const int2 b = pw[((rd.n_e + rd.n_k - 1 + (1 << lg) - 1) >> lg) + s0];
    idx = (uint32_t)b.x;
    k += b.y;
  }
  const int cg = min(64, EXPAND_BANDS >> lg); /* groups per chunk */
  const int gs = s0 * sl;
  int2 w = make_int2(0, 0);
  if (lane < cg && gs + lane < g1) w = pw[gs + lane];
  for (int g = gs; g < g1; g += cg) {
    uint32_t V = (uint32_t)w.x;
    const uint32_t M = (uint32_t)w.y;
    w = make_int2(0, 0);
    if (lane < cg && g + cg + lane < g1) w = pw[g + cg + lane]; /* the next chunk's */
    /* at most 1024 cells a chunk: both counts scanned in one word */
    const uint32_t n = (uint32_t)__popc(V) | ((uint32_t)__popc(M) << 16);
    const uint32_t inc = lane_scan(n);
    const uint32_t all = rlane_u(inc, 63);
    const uint32_t exc = inc - n;
    uint32_t at = exc & 0xffffu;
    int kk = k + (int)(exc >> 16);
    const int t0 = (g + lane) << lg;
    while (V) {
      const int b = __ffs(V) - 1;
      V &= V - 1;
      kk += (int)((M >> b) & 1u);
      cell[at++] = make_int2(t0 + b - kk, kk);
    }
    __syncthreads();
    const uint32_t cnt = all & 0xffffu;
    for (uint32_t p = lane; p < cnt; p += 64) out[idx + p] = cell[p];
    __syncthreads();
    idx += cnt;
    k += (int)(all >> 16);
  }
}

/* ------------------------------------------------------------- launchers */

hipError_t launch_prep(const ReadDesc *reads, int n_planned, const float *events, int ev_stride,
                       const uint32_t *ranks, const uint64_t *in_addr, const float *scale,
                       const float *shift, bool scale_events, float *xmean, uint32_t *krank,
                       int32_t *rstat, uint32_t *queue, hipStream_t st) {
  if (n_planned <= 0) return hipSuccess;
  /* one wavefront per read when there is nothing to stage */
  const int threads = (xmean || krank) ? 256 : 64;
  hipLaunchKernelGGL(k_prep, dim3(n_planned), dim3(threads), 0, st, reads, events, ev_stride, ranks, in_addr,
                     scale, shift, (int)scale_events, xmean, krank, rstat, queue);
  return hipGetLastError();
}

/* Kernel variants: (slots per lane, refills per group, CLEAR of band_read).  At
 * two and four slots per lane the kernels run interior bands in abea_interior.h,
 * ec = 1 + W mod cpl; where its refill intervals do not fit (W = 252 at four: see
 * interior_refills), and at other slot counts, the window kernels run (ec = 0). */
#define ABEA_VARIANTS(CALL)                             \
  if (cpl == 1 && rpg == 1 && !ec) CALL(1, 1, 0);       \
  if (cpl == 1 && rpg == 2 && !ec) CALL(1, 2, 0);       \
  if (cpl == 2 && rpg == 1 && ec == 1) CALL(2, 1, 1);   \
  if (cpl == 2 && rpg == 1 && ec == 2) CALL(2, 1, 2);   \
  if (cpl == 2 && rpg == 2 && ec == 1) CALL(2, 2, 1);   \
  if (cpl == 2 && rpg == 2 && ec == 2) CALL(2, 2, 2);   \
  if (cpl == 2 && rpg == 4 && ec == 1) CALL(2, 4, 1);   \
  if (cpl == 4 && rpg == 1 && ec == 1) CALL(4, 1, 1);   \
  if (cpl == 4 && rpg == 1 && ec == 2) CALL(4, 1, 2);   \
  if (cpl == 4 && rpg == 1 && ec == 3) CALL(4, 1, 3);   \
  if (cpl == 4 && rpg == 1 && ec == 4) CALL(4, 1, 4);   \
  if (cpl == 4 && rpg == 2 && ec == 0) CALL(4, 2, 0);   \
  if (cpl == 4 && rpg == 2 && ec == 1) CALL(4, 2, 1);   \
  if (cpl == 4 && rpg == 2 && ec == 2) CALL(4, 2, 2);   \
  if (cpl == 4 && rpg == 2 && ec == 3) CALL(4, 2, 3);   \
  if (cpl == 4 && rpg == 2 && ec == 4) CALL(4, 2, 4);   \
  if (cpl == 4 && rpg == 4 && ec == 3) CALL(4, 4, 3);   \
  if (cpl == 4 && rpg == 4 && ec == 4) CALL(4, 4, 4);   \
  if (cpl == 8 && rpg == 1 && !ec) CALL(8, 1, 0);       \
  if (cpl == 8 && rpg == 2 && !ec) CALL(8, 2, 0);       \
  if (cpl == 16 && rpg == 1 && !ec) CALL(16, 1, 0);

static void variant(int cpl, int W, int &rpg, int &ec) {
  rpg = interior_refills(W, cpl);
  ec = rpg > 0 ? 1 + W % cpl : 0;
  if (rpg == 0) rpg = refills_per_group(W, cpl);
}

hipError_t launch_band(const AlignArgs &a, int cpl, hipStream_t st, hipEvent_t t0,
                       hipEvent_t t1) {
  if (a.n_reads <= 0) return hipSuccess;
  int rpg, ec;
  variant(cpl, a.W, rpg, ec);
#define ABEA_L(C, R, E)                                                                                 \
  {                                                                                                     \
    if (a.trim)                                                                                         \
      hipExtLaunchKernelGGL((k_band<C, R, E, true>), dim3(a.n_reads), dim3(64), 0, st, t0, t1, 0, a);  \
    else                                                                                                \
      hipExtLaunchKernelGGL((k_band<C, R, E, false>), dim3(a.n_reads), dim3(64), 0, st, t0, t1, 0, a); \
    return hipGetLastError();                                                                           \
  }
  ABEA_VARIANTS(ABEA_L)
#undef ABEA_L
  return hipErrorInvalidValue;
}

template <bool TRIM>
static hipError_t launch_backtrack_t(const AlignArgs &a, int cpl, hipStream_t st) {
  switch (cpl) {
    case 1: hipLaunchKernelGGL((k_backtrack<1, TRIM>), dim3(a.n_reads), dim3(64), 0, st, a); break;
    case 2: hipLaunchKernelGGL((k_backtrack<2, TRIM>), dim3(a.n_reads), dim3(64), 0, st, a); break;
    case 4: hipLaunchKernelGGL((k_backtrack<4, TRIM>), dim3(a.n_reads), dim3(64), 0, st, a); break;
    case 8: hipLaunchKernelGGL((k_backtrack<8, TRIM>), dim3(a.n_reads), dim3(64), 0, st, a); break;
    case 16: hipLaunchKernelGGL((k_backtrack<16, TRIM>), dim3(a.n_reads), dim3(64), 0, st, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_backtrack(const AlignArgs &a, int cpl, hipStream_t st) {
  if (a.n_reads <= 0) return hipSuccess;
  return a.trim ? launch_backtrack_t<true>(a, cpl, st) : launch_backtrack_t<false>(a, cpl, st);
}

template <int CPL, int RPG, int EDGE, bool TRIM>
static hipError_t launch_align_c(const AlignArgs &a, int wpg, hipStream_t st, hipEvent_t t0,
                                 hipEvent_t t1) {
  const dim3 grid((a.n_workers + wpg - 1) / wpg);
  switch (wpg) {
    case 1: hipExtLaunchKernelGGL((k_align<CPL, RPG, 1, EDGE, TRIM>), grid, dim3(64), 0, st, t0, t1, 0, a); break;
    case 2: hipExtLaunchKernelGGL((k_align<CPL, RPG, 2, EDGE, TRIM>), grid, dim3(128), 0, st, t0, t1, 0, a); break;
    case 4: hipExtLaunchKernelGGL((k_align<CPL, RPG, 4, EDGE, TRIM>), grid, dim3(256), 0, st, t0, t1, 0, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_align(const AlignArgs &a, int cpl, int wpg, hipStream_t st,
                        hipEvent_t t0, hipEvent_t t1) {
  if (a.n_reads <= 0 || a.n_workers <= 0) return hipSuccess;
  if (a.n_workers > a.n_reads) return hipErrorInvalidValue;
  int rpg, ec;
  variant(cpl, a.W, rpg, ec);
#define ABEA_L(C, R, E)                                                                                       \
  return a.trim ? launch_align_c<C, R, E, true>(a, wpg, st, t0, t1) : launch_align_c<C, R, E, false>(a, wpg, st, t0, t1)
  ABEA_VARIANTS(ABEA_L)
#undef ABEA_L
  return hipErrorInvalidValue;
}

template <int CPL, int RPG, int EDGE, bool TRIM>
static int groups_per_cu_c(int wpg) {
  int n = 0;
  hipError_t e = hipErrorInvalidValue;
  switch (wpg) {
    case 1: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_align<CPL, RPG, 1, EDGE, TRIM>, 64, 0); break;
    case 2: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_align<CPL, RPG, 2, EDGE, TRIM>, 128, 0); break;
    case 4: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_align<CPL, RPG, 4, EDGE, TRIM>, 256, 0); break;
  }
  /* the runtime counts the registers used, not the room most_per_simd leaves */
  return e == hipSuccess ? std::min(n, 4 * most_per_simd(CPL, TRIM) / wpg) : 0;
}

int align_groups_per_cu(int cpl, int wpg, bool trim, int W) {
  int rpg, ec;
  variant(cpl, W, rpg, ec);
#define ABEA_L(C, R, E) return trim ? groups_per_cu_c<C, R, E, true>(wpg) : groups_per_cu_c<C, R, E, false>(wpg)
  ABEA_VARIANTS(ABEA_L)
#undef ABEA_L
  return 0;
}

/* the plan from mapped pinned host memory into device memory, one thread per
 * read */
__global__ __launch_bounds__(256) void k_stage_plan(const ReadDesc *__restrict__ src, ReadDesc *__restrict__ dst,
                                                    int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

hipError_t launch_stage_plan(const ReadDesc *src, ReadDesc *dst, int n, hipStream_t st) {
  if (n > 0) hipLaunchKernelGGL(k_stage_plan, dim3((n + 255) / 256), dim3(256), 0, st, src, dst, n);
  return hipGetLastError();
}

hipError_t launch_scan(const uint64_t *len, int n, uint64_t *offset, hipStream_t st) {
  hipLaunchKernelGGL(k_scan, dim3(1), dim3(64), 0, st, len, n, offset);
  return hipGetLastError();
}

hipError_t launch_expand(const ReadDesc *reads, int n, int cpl, const int2 *scratch, const uint64_t *path_src,
                         const uint64_t *offset, int2 *pairs, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  /* eight wavefronts per read, up to one per segment where the reads are
   * few: 100 reads of up to 1 Mb take 607 us at eight */
  const int split = std::min(WALK_MAX_SEGMENTS, std::max(8, 16384 / n));
  hipLaunchKernelGGL(k_expand, dim3(n, split), dim3(64), 0, st, reads, scratch, path_src, offset,
                     __builtin_ctz((unsigned)bands_per_group(cpl)), pairs);
  return hipGetLastError();
}

/* ------------------------------------------------ fixed device scratch */

/* Scratch of the no-allocation entry point: one array per device, held from
 * the library's load until the process ends.  Host code must not pass this
 * name to a kernel or a copy (in host code it is a host-side stand-in, not a
 * device address); it uses the address noalloc_scratch() returns. */
static __device__ __align__(256) unsigned char scratch[NOALLOC_SCRATCH_BYTES];

hipError_t noalloc_scratch(int device, void **ptr) {
  /* hipGetSymbolAddress once per device, with that device current (the
   * caller has made it current), kept for the life of the process */
  static std::mutex mu;
  static void *addr[NOALLOC_MAX_DEVICES] = {};
  *ptr = nullptr;
  if (device < 0 || device >= NOALLOC_MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(mu);
  if (!addr[device]) {
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[device] = p;
  }
  *ptr = addr[device];
  return hipSuccess;
}

}  // namespace abea
