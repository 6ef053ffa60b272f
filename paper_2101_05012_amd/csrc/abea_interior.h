/*
 * abea_interior.h -- the interior bands of the band fill at two and four slots
 * per lane (see band_read in abea_kernels.hip): a refill interval of bands that
 * lie wholly inside the DP table, in gfx950 assembly.
 *
 * What bounds a band.  With several wavefronts on a SIMD it starts about one
 * instruction per two cycles, vector or scalar (20000 uneven reads at W = 100:
 * 49 instructions and 101 cycles per band as compiled), and a lane rotation
 * or v_readlane holds the vector unit for four cycles in which no other
 * wavefront starts; a lone wavefront starts one instruction per four cycles
 * (five where it is eight bytes long) and waits 16 more where the scalar unit
 * reads what the vector unit wrote.  Either way the count of instructions
 * decides.  Of the band's 49, 28 made its 128 cells; most of the others found
 * the registers of its first, last and cleared slots, which depend on
 * (first k-mer K) mod CPL and change with every k-mer move, and carried masks
 * and indices for them.
 *
 * So the code is laid out by state: the band is written once for every value
 * of K mod CPL (registers fixed in the text) and every band of the interval, and
 * a k-mer move is a branch to the next band's code for the next state.  What
 * remains of a move is one bit test and that branch.  Lane numbers are kept in
 * scalar registers as K div CPL and constant distances from it, which change
 * only when K mod CPL wraps.  In an interval a lane's slots hold CPL consecutive
 * k-mers from a multiple of CPL, so their events are a window that slides by one
 * event a band: one LDS word per lane and band feeds all its slots.  Per band at
 * two slots per lane: 32 vector instructions, 2 scalar and half an LDS read,
 * where the compiled form had 35, 12 and 1; at four slots 60, 2 and 1.
 *
 * A band, with P the scores of band i-2 and Q of band i-1 (band i replaces P):
 *   - scores (Alg. 5.2): diagonal + step, up + stay and left + skip, plus the
 *     emission, the first two rounded as (pred + lp) + em; v_max3.  The rotated
 *     neighbours of register 0 (LF: left + skip, DG: diagonal + step) were made
 *     at the end of the band before;
 *   - the slots beside the band (k-mers K-1 and K+W) are cleared by
 *     v_writelane: the quiet NaN of the inline constant -1, which v_max3 passes
 *     over as it would -inf, and which equals no candidate.  Every cell of the
 *     band is finite (the caller brings no event or k-mer here that could make
 *     another), so one of v_max3's operands always is a number;
 *   - the move: the band's first cell against its last (v_readlane, then one
 *     compare against every lane, whose bit for the last cell's lane decides;
 *     both are finite, so the alternation for two cells of -inf is not here).
 *     With other wavefronts on the SIMD the rotations for the next band and the
 *     v_readlane run at raised priority: wavefronts waiting at such an
 *     instruction pass it first and the others find partners to start beside
 *     (20000 uneven reads, W = 100: 80 ms a pass against 91 without).  The
 *     longest reads of a batch run at a higher priority throughout instead, and
 *     a lone wavefront saves the two instructions;
 *   - trace bits: two compares and shift-ins per register, through VCC; the two
 *     wait states between a compare and the shift-in that reads it are filled
 *     with the next band's emission (Alg. 5.3), c - ((x - mu')^2 * h).
 * Measured as a whole, compiled -> this, with the same walk: 20000 uneven reads
 * at W = 100 96.8 -> 77.0 ms, 10000 at W = 200 134 -> 97.0 ms, 100 of up to 1 Mb
 * (one lone wavefront's chain) 303 -> 248 ms, 64 of 1 kb 365 -> 342 us.
 * Wait states kept: 2 from a VALU write of VCC or an SGPR to its VALU read, 2
 * from a VGPR write to its DPP read, 1 to its v_readlane.
 */
#ifndef ABEA_INTERIOR_H
#define ABEA_INTERIOR_H

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace abea {

/* What a refill interval of interior bands works on.  p and q: the scores of the
 * two bands before it (p the older), afterwards of its last two.  K: the first
 * k-mer of its first band (that band's move applied), afterwards of its last;
 * mv: the move after that one (1: a k-mer move). */
template <int CPL>
struct Interior {
  float p[CPL], q[CPL];
  uint32_t td, tu;   /* trace words */
  float lf, dg;      /* register 0's left + skip and diagonal + step for the next band */
  uint32_t ak;       /* LDS byte address of the parameters (mu', c, h, pad) of the lane's first k-mer */
  uint32_t ax;       /* LDS byte address of the event of its last k-mer at the first band (see below) */
  float stay, skip, step;
  int K, mv;
  int calm;          /* 1: priority raised only where instructions start alone; 0: one of the longest reads */
};

/* The macros below are the assembler's, named by the statement's own number.
 *
 * Both forms are in one statement, z = 1 the one that raises its priority, z = 0
 * for the longest reads.  move: r, h the registers of the first and last cell, lo
 * the first's lane; pt, qt the top registers of the two bands, rotated for the next
 * band. */
#define ABEA_ASM_COMMON R"(
.macro move%= z, r, h, lo, pt, qt
.if \z
  s_setprio 1
.endif
  v_readlane_b32 %[lo], \r, \lo
  v_add_f32_dpp %[dg], \qt, %[step] wave_ror:1 row_mask:0xf bank_mask:0xf
  v_add_f32_dpp %[lf], \pt, %[skip] wave_ror:1 row_mask:0xf bank_mask:0xf
.if \z
  s_setprio 0
.endif
  v_cmp_lt_f32_e64 %[cm], %[lo], \h
.endm
.macro em1%= e, x, m, f, y, n
  v_sub_f32_e32 \e, \x, \m
  v_sub_f32_e32 \f, \y, \n
.endm
.macro em2%= e, f
  v_mul_f32_e32 \e, \e, \e
  v_mul_f32_e32 \f, \f, \f
.endm
.macro em3%= e, h, f, i
  v_mul_f32_e32 \e, \h, \e
  v_mul_f32_e32 \f, \i, \f
.endm
.macro em4%= e, c, f, d
  v_sub_f32_e32 \e, \c, \e
  v_sub_f32_e32 \f, \d, \f
.endm
.macro bit1%= p, s
  v_cmp_eq_f32_e32 vcc, \p, \s
.endm
.macro bit2%= t
  v_addc_co_u32_e32 \t, vcc, \t, \t, vcc
.endm
.macro slow%= p, d, u
  bit1%= \p, \d
  s_nop 1
  bit2%= %[td]
  bit1%= \p, \u
  s_nop 1
  bit2%= %[tu]
.endm
)"

/* ------------------------------------------------- two slots per lane */

/* band2 s, b, n, p, q, ...: band b of the interval in state s (K mod 2); n =
 * b+1; x, y the next band's events of registers 0 and 1 (wt: wait for their
 * read); rd >= 0: then read events rd and rd+1 of the window into xr (event 0 is
 * register 1's in band 0, and in band b registers 0 and 1 take events b+1 and
 * b); r, h, lo, hi the registers and lanes of the first and last cell; c1/l1, c2/l2
 * the cleared registers and lanes (not r last: v_readlane follows); mv the next
 * band's code after a k-mer move.  end2: the interval's last band.  v[4:5] and
 * v[6:7] hold the window, v[8:10] and v[12:14] the two k-mers' parameters. */
#define ABEA_ASM2 R"(
.macro core2%= z, p0, p1, q0, q1, r, h, c1, l1, c2, l2, lo
  v_add_f32_e32 %[t0], %[stay], \q0
  v_add_f32_e32 %[t1], %[stay], \q1
  v_add_f32_e32 %[t2], %[skip], \q0
  v_add_f32_e32 %[t3], %[step], \p0
  v_add_f32_e32 %[t4], %[dg], %[e0]
  v_add_f32_e32 %[t0], %[t0], %[e0]
  v_add_f32_e32 %[t3], %[t3], %[e1]
  v_add_f32_e32 %[t1], %[t1], %[e1]
  v_max3_f32 \p1, %[t3], %[t1], %[t2]
  v_max3_f32 \p0, %[t4], %[t0], %[lf]
  v_writelane_b32 \c1, -1, \l1
  v_writelane_b32 \c2, -1, \l2
  move%= \z, \r, \h, \lo, \p1, \q1
.endm
.macro band2%= z, s, b, n, p0, p1, q0, q1, x, y, wt, rd, xr, r, h, c1, l1, c2, l2, lo, hi, mv
.Lb\z\s\()_\b\()_%=:
  core2%= \z, \p0, \p1, \q0, \q1, \r, \h, \c1, \l1, \c2, \l2, \lo
.if \wt
  s_waitcnt lgkmcnt(0)
.endif
  bit1%= \p0, %[t4]
  em1%= %[e0], \x, v8, %[e1], \y, v12
  bit2%= %[td]
.if \rd >= 0
  ds_read2_b32 \xr, %[ax] offset0:\rd offset1:\rd+1
.endif
  bit1%= \p0, %[t0]
  em2%= %[e0], %[e1]
  bit2%= %[tu]
  bit1%= \p1, %[t3]
  em3%= %[e0], v10, %[e1], v14
  bit2%= %[td]
  bit1%= \p1, %[t1]
  em4%= %[e0], v9, %[e1], v13
  bit2%= %[tu]
  s_bitcmp1_b64 %[cm], \hi
  s_cbranch_scc1 \mv\()_\n\()_%=
.endm
.macro end2%= z, s, b, p0, p1, q0, q1, r, h, c1, l1, c2, l2, lo, hi
.Lb\z\s\()_\b\()_%=:
  core2%= \z, \p0, \p1, \q0, \q1, \r, \h, \c1, \l1, \c2, \l2, \lo
  slow%= \p0, %[t4], %[t0]
  slow%= \p1, %[t3], %[t1]
  s_lshl_b32 %[K], %[la], 1
  s_or_b32 %[K], %[K], \s
  s_bitcmp1_b64 %[cm], \hi
  s_cselect_b32 %[mv], 1, 0
.if \s + \z < 2
  s_branch .Lend_%=
.endif
.endm
.macro wrap2%= z, b
.Lw\z\()_\b\()_%=:
  s_add_u32 %[la], %[la], 1
  s_add_u32 %[lb], %[lb], 1
  s_add_u32 %[lc], %[lc], 1
  s_add_u32 %[ld], %[ld], 1
  s_branch .Lb\z\()0_\b\()_%=
.endm
  ds_read_b96 v[8:10], %[ak]
  ds_read_b96 v[12:14], %[ak] offset:16
  ds_read2_b32 v[4:5], %[ax] offset0:0 offset1:1
  ds_read2_b32 v[6:7], %[ax] offset0:2 offset1:3
  s_lshl1_add_u32 %[lo], %[K], %[calm]
  s_and_b32 %[lo], %[lo], 3
  s_waitcnt lgkmcnt(0)
  em1%= %[e0], v5, v8, %[e1], v4, v12
  em2%= %[e0], %[e1]
  em3%= %[e0], v10, %[e1], v14
  em4%= %[e0], v9, %[e1], v13
  s_cmp_eq_u32 %[lo], 0
  s_cbranch_scc1 .Lb00_0_%=
  s_cmp_eq_u32 %[lo], 2
  s_cbranch_scc1 .Lb01_0_%=
  s_cmp_eq_u32 %[lo], 3
  s_cbranch_scc1 .Lb11_0_%=
  s_branch .Lb10_0_%=
)"

/* The states of K mod 2.  la = K div 2, lb = la-1, lc = la+h; W even (h = W/2):
 * ld = la+h-1; W odd (h = W div 2): ld = la+h+1. */
#define ABEA_P2 "%[p0], %[p1], %[q0], %[q1], "
#define ABEA_Q2 "%[q0], %[q1], %[p0], %[p1], "
#define ABEA_E0(A, B) A ", " B ", " A ", %[lc], " B ", %[lb], %[la], %[ld]"
#define ABEA_E1(A, B) B ", " A ", " B ", %[lc], " A ", %[la], %[la], %[lc]"
#define ABEA_O0(A, B) A ", " A ", " B ", %[lb], " B ", %[lc], %[la], %[lc]"
#define ABEA_O1(A, B) B ", " B ", " A ", %[la], " A ", %[ld], %[la], %[lc]"
/* bands B (even) and B+1: two events of the window come from the pair CUR, two
 * from NEXT, whose read band B waits for (WT) before it reads events RD into CUR */
#define ABEA_PAIR2(Z, S, ST, MV, B, B1, B2, CUR, C1, N0, N1, WT, RD)                                             \
  "band2%= " #Z ", " #S ", " #B ", " #B1 ", " ABEA_P2 #N0 ", " #C1 ", " #WT ", " #RD ", " CUR ", "                    \
             ST("%[p0]", "%[p1]") ", " MV "\n"                                                                \
  "band2%= " #Z ", " #S ", " #B1 ", " #B2 ", " ABEA_Q2 #N1 ", " #N0 ", 0, -1, " CUR ", " ST("%[q0]", "%[q1]") ", " MV "\n"
#define ABEA_LAST2(Z, S, ST, MV, B, B1, C1, N0, WT)                                                              \
  "band2%= " #Z ", " #S ", " #B ", " #B1 ", " ABEA_P2 #N0 ", " #C1 ", " #WT ", -1, v[4:5], " ST("%[p0]", "%[p1]") ", " MV "\n" \
  "end2%= " #Z ", " #S ", " #B1 ", " ABEA_Q2 ST("%[q0]", "%[q1]") "\n"
#define ABEA_ROW2_4(Z, S, ST, MV) \
  ABEA_PAIR2(Z, S, ST, MV, 0, 1, 2, "v[4:5]", v5, v6, v7, 0, 4) ABEA_LAST2(Z, S, ST, MV, 2, 3, v7, v4, 1)
#define ABEA_ROW2_6(Z, S, ST, MV)                                  \
  ABEA_PAIR2(Z, S, ST, MV, 0, 1, 2, "v[4:5]", v5, v6, v7, 0, 4)    \
  ABEA_PAIR2(Z, S, ST, MV, 2, 3, 4, "v[6:7]", v7, v4, v5, 1, 6)    \
  ABEA_PAIR2(Z, S, ST, MV, 4, 5, 6, "v[4:5]", v5, v6, v7, 1, 8)
#define ABEA_ROW2_8(Z, S, ST, MV) ABEA_ROW2_6(Z, S, ST, MV) ABEA_LAST2(Z, S, ST, MV, 6, 7, v7, v4, 1)
#define ABEA_ROW2_16(Z, S, ST, MV)                                                                                   \
  ABEA_ROW2_6(Z, S, ST, MV) ABEA_PAIR2(Z, S, ST, MV, 6, 7, 8, "v[6:7]", v7, v4, v5, 1, 10)                              \
  ABEA_PAIR2(Z, S, ST, MV, 8, 9, 10, "v[4:5]", v5, v6, v7, 1, 12)                                                    \
  ABEA_PAIR2(Z, S, ST, MV, 10, 11, 12, "v[6:7]", v7, v4, v5, 1, 14)                                                  \
  ABEA_PAIR2(Z, S, ST, MV, 12, 13, 14, "v[4:5]", v5, v6, v7, 1, 16) ABEA_LAST2(Z, S, ST, MV, 14, 15, v7, v4, 1)
#define ABEA_WRAP2_4(Z) "wrap2%= " #Z ", 1\n wrap2%= " #Z ", 2\n wrap2%= " #Z ", 3\n"
#define ABEA_WRAP2_8(Z)                                                                            \
  ABEA_WRAP2_4(Z) "wrap2%= " #Z ", 4\n wrap2%= " #Z ", 5\n wrap2%= " #Z ", 6\n wrap2%= " #Z ", 7\n"
#define ABEA_WRAP2_16(Z)                                                                           \
  ABEA_WRAP2_8(Z) "wrap2%= " #Z ", 8\n wrap2%= " #Z ", 9\n wrap2%= " #Z ", 10\n wrap2%= " #Z    \
                  ", 11\n wrap2%= " #Z ", 12\n wrap2%= " #Z ", 13\n wrap2%= " #Z ", 14\n wrap2%= " #Z ", 15\n"
/* the rows that run into the end come last, the wrap entries first */
#define ABEA_RUN2(ROW, WRAP, S0, S1)                                                                  \
  asm(ABEA_ASM_COMMON ABEA_ASM2 WRAP(0) WRAP(1) ROW(0, 0, S0, ".Lb01") ROW(0, 1, S1, ".Lw0")                     \
          ROW(1, 0, S0, ".Lb11") ROW(1, 1, S1, ".Lw1") ".Lend_%=:\n"                                            \
      : [p0] "+v"(v.p[0]), [p1] "+v"(v.p[1]), [q0] "+v"(v.q[0]), [q1] "+v"(v.q[1]), [td] "+v"(v.td),             \
        [tu] "+v"(v.tu), [lf] "+v"(v.lf), [dg] "+v"(v.dg), [e0] "=&v"(e0), [e1] "=&v"(e1), [t0] "=&v"(t0),       \
        [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3), [t4] "=&v"(t4), [lo] "=&s"(lo), [cm] "=&s"(cm),          \
        [mv] "=&s"(v.mv), [K] "+&s"(v.K), [la] "+&s"(la), [lb] "+&s"(lb), [lc] "+&s"(lc), [ld] "+&s"(ld)         \
      : [ak] "v"(v.ak), [ax] "v"(v.ax), [calm] "s"(v.calm), [stay] "v"(v.stay), [skip] "v"(v.skip), [step] "v"(v.step) \
      : "v4", "v5", "v6", "v7", "v8", "v9", "v10", "v12", "v13", "v14", "vcc", "scc", "memory")

/* NB interior bands (4, 8 or 16) at two slots per lane; M = W mod 2. */
template <int NB, int M>
__device__ __forceinline__ void interior(Interior<2> &v, int W) {
  float e0, e1, t0, t1, t2, t3, t4;
  uint64_t cm;
  int lo, la = v.K >> 1, lb = la - 1, lc = la + (W >> 1), ld = M == 0 ? lc - 1 : lc + 1;
  static_assert(NB == 4 || NB == 8 || NB == 16, "a refill interval of 4, 8 or 16 bands");
  if constexpr (NB == 16 && M == 0)
    ABEA_RUN2(ABEA_ROW2_16, ABEA_WRAP2_16, ABEA_E0, ABEA_E1);
  else if constexpr (NB == 16)
    ABEA_RUN2(ABEA_ROW2_16, ABEA_WRAP2_16, ABEA_O0, ABEA_O1);
  else if constexpr (NB == 8 && M == 0)
    ABEA_RUN2(ABEA_ROW2_8, ABEA_WRAP2_8, ABEA_E0, ABEA_E1);
  else if constexpr (NB == 8)
    ABEA_RUN2(ABEA_ROW2_8, ABEA_WRAP2_8, ABEA_O0, ABEA_O1);
  else if constexpr (M == 0)
    ABEA_RUN2(ABEA_ROW2_4, ABEA_WRAP2_4, ABEA_E0, ABEA_E1);
  else
    ABEA_RUN2(ABEA_ROW2_4, ABEA_WRAP2_4, ABEA_O0, ABEA_O1);
}

/* ------------------------------------------------ four slots per lane */

/* As at two; K mod 4 and W mod 4 choose the registers, h = W div 4.  Event 0 of
 * the window is register 3's in band 0; in band b register c takes event b+3-c.
 * The ring's event e lies in sub-ring e mod 4 (EVENT_SUBRING words long) at entry
 * e div 4; res is event 0's sub-ring and ax its entry in sub-ring 0.  v4, v5,
 * v6, v7 and v11 hold the window (event j in the (j mod 5)th), v[8:10], v[12:14],
 * v[16:18] and v[20:22] the k-mers' parameters. */
constexpr int EVENT_SUBRING = 130;
#define ABEA_ASM4 R"(
.macro read4%= x, j
  ds_read_b32 \x, %[ax] offset:(((\j+res%=)&3)*130+((\j+res%=)>>2))*4
.endm
.macro core4%= z, p0, p1, p2, p3, q0, q1, q2, q3, r, h, c1, l1, c2, l2
  v_add_f32_e32 %[t0], %[stay], \q0
  v_add_f32_e32 %[t1], %[stay], \q1
  v_add_f32_e32 %[t2], %[stay], \q2
  v_add_f32_e32 %[t3], %[stay], \q3
  v_add_f32_e32 %[t4], %[skip], \q0
  v_add_f32_e32 %[t5], %[skip], \q1
  v_add_f32_e32 %[t6], %[skip], \q2
  v_add_f32_e32 %[t7], %[step], \p0
  v_add_f32_e32 %[t8], %[step], \p1
  v_add_f32_e32 %[t9], %[step], \p2
  v_add_f32_e32 %[ta], %[dg], %[e0]
  v_add_f32_e32 %[t0], %[t0], %[e0]
  v_add_f32_e32 %[t7], %[t7], %[e1]
  v_add_f32_e32 %[t1], %[t1], %[e1]
  v_add_f32_e32 %[t8], %[t8], %[e2]
  v_add_f32_e32 %[t2], %[t2], %[e2]
  v_add_f32_e32 %[t9], %[t9], %[e3]
  v_add_f32_e32 %[t3], %[t3], %[e3]
  v_max3_f32 \p3, %[t9], %[t3], %[t6]
  v_max3_f32 \p2, %[t8], %[t2], %[t5]
  v_max3_f32 \p1, %[t7], %[t1], %[t4]
  v_max3_f32 \p0, %[ta], %[t0], %[lf]
  v_writelane_b32 \c1, -1, \l1
  v_writelane_b32 \c2, -1, \l2
  move%= \z, \r, \h, %[la], \p3, \q3
.endm
.macro band4%= z, s, b, n, p0, p1, p2, p3, q0, q1, q2, q3, x3, x2, x1, x0, rd, xr, r, h, hi, c1, l1, c2, l2, mv
.Lb\z\s\()_\b\()_%=:
  core4%= \z, \p0, \p1, \p2, \p3, \q0, \q1, \q2, \q3, \r, \h, \c1, \l1, \c2, \l2
.if \b
  s_waitcnt lgkmcnt(0)
.endif
  bit1%= \p0, %[ta]
  em1%= %[e0], \x0, v8, %[e1], \x1, v12
  bit2%= %[td]
.if \rd >= 0
  read4%= \xr, \rd
.endif
  bit1%= \p0, %[t0]
  em1%= %[e2], \x2, v16, %[e3], \x3, v20
  bit2%= %[tu]
  bit1%= \p1, %[t7]
  em2%= %[e0], %[e1]
  bit2%= %[td]
  bit1%= \p1, %[t1]
  em2%= %[e2], %[e3]
  bit2%= %[tu]
  bit1%= \p2, %[t8]
  em3%= %[e0], v10, %[e1], v14
  bit2%= %[td]
  bit1%= \p2, %[t2]
  em3%= %[e2], v18, %[e3], v22
  bit2%= %[tu]
  bit1%= \p3, %[t9]
  em4%= %[e0], v9, %[e1], v13
  bit2%= %[td]
  bit1%= \p3, %[t3]
  em4%= %[e2], v17, %[e3], v21
  bit2%= %[tu]
  s_bitcmp1_b64 %[cm], \hi
  s_cbranch_scc1 \mv\()_\n\()_%=
.endm
.macro end4%= z, s, b, p0, p1, p2, p3, q0, q1, q2, q3, r, h, hi, c1, l1, c2, l2
.Lb\z\s\()_\b\()_%=:
  core4%= \z, \p0, \p1, \p2, \p3, \q0, \q1, \q2, \q3, \r, \h, \c1, \l1, \c2, \l2
  slow%= \p0, %[ta], %[t0]
  slow%= \p1, %[t7], %[t1]
  slow%= \p2, %[t8], %[t2]
  slow%= \p3, %[t9], %[t3]
  s_lshl_b32 %[K], %[la], 2
  s_or_b32 %[K], %[K], \s
  s_bitcmp1_b64 %[cm], \hi
  s_cselect_b32 %[mv], 1, 0
.if \s + \z < 4
  s_branch .Lend_%=
.endif
.endm
.macro wrap4%= z, b
.Lw\z\()_\b\()_%=:
  s_add_u32 %[la], %[la], 1
  s_add_u32 %[lb], %[lb], 1
  s_add_u32 %[lc], %[lc], 1
  s_add_u32 %[ld], %[ld], 1
  s_add_u32 %[le], %[le], 1
  s_branch .Lb\z\()0_\b\()_%=
.endm
  ds_read_b96 v[8:10], %[ak]
  ds_read_b96 v[12:14], %[ak] offset:16
  ds_read_b96 v[16:18], %[ak] offset:32
  ds_read_b96 v[20:22], %[ak] offset:48
  read4%= v4, 0
  read4%= v5, 1
  read4%= v6, 2
  read4%= v7, 3
  read4%= v11, 4
  s_and_b32 %[lo], %[K], 3
  s_lshl1_add_u32 %[lo], %[lo], %[calm]
  s_waitcnt lgkmcnt(0)
  em1%= %[e0], v7, v8, %[e1], v6, v12
  em1%= %[e2], v5, v16, %[e3], v4, v20
  em2%= %[e0], %[e1]
  em2%= %[e2], %[e3]
  em3%= %[e0], v10, %[e1], v14
  em3%= %[e2], v18, %[e3], v22
  em4%= %[e0], v9, %[e1], v13
  em4%= %[e2], v17, %[e3], v21
  s_cmp_eq_u32 %[lo], 0
  s_cbranch_scc1 .Lb00_0_%=
  s_cmp_eq_u32 %[lo], 1
  s_cbranch_scc1 .Lb10_0_%=
  s_cmp_eq_u32 %[lo], 2
  s_cbranch_scc1 .Lb01_0_%=
  s_cmp_eq_u32 %[lo], 3
  s_cbranch_scc1 .Lb11_0_%=
  s_cmp_eq_u32 %[lo], 4
  s_cbranch_scc1 .Lb02_0_%=
  s_cmp_eq_u32 %[lo], 5
  s_cbranch_scc1 .Lb12_0_%=
  s_cmp_eq_u32 %[lo], 6
  s_cbranch_scc1 .Lb03_0_%=
  s_branch .Lb13_0_%=
)"

/* State s of K mod 4 for W mod 4 = m: the registers of the first and last cell,
 * the last's lane, the cleared registers and lanes (k-mer K+W, then K-1).  The
 * first cell's lane is la = K div 4; lb = la-1, lc = la+h, ld = la+h+1, le = la+h-1. */
#define ABEA_P4 "%[p0], %[p1], %[p2], %[p3], %[q0], %[q1], %[q2], %[q3], "
#define ABEA_Q4 "%[q0], %[q1], %[q2], %[q3], %[p0], %[p1], %[p2], %[p3], "
#define ABEA_S4(R, H, HL, C1, L1, C2, L2, A) \
  "%[" A #R "], %[" A #H "], %[" #HL "], %[" A #C1 "], %[" #L1 "], %[" A #C2 "], %[" #L2 "]"
#define ABEA_W0_0(A) ABEA_S4(0, 3, le, 0, lc, 3, lb, A)
#define ABEA_W0_1(A) ABEA_S4(1, 0, lc, 1, lc, 0, la, A)
#define ABEA_W0_2(A) ABEA_S4(2, 1, lc, 2, lc, 1, la, A)
#define ABEA_W0_3(A) ABEA_S4(3, 2, lc, 3, lc, 2, la, A)
#define ABEA_W1_0(A) ABEA_S4(0, 0, lc, 1, lc, 3, lb, A)
#define ABEA_W1_1(A) ABEA_S4(1, 1, lc, 2, lc, 0, la, A)
#define ABEA_W1_2(A) ABEA_S4(2, 2, lc, 3, lc, 1, la, A)
#define ABEA_W1_3(A) ABEA_S4(3, 3, lc, 0, ld, 2, la, A)
#define ABEA_W2_0(A) ABEA_S4(0, 1, lc, 2, lc, 3, lb, A)
#define ABEA_W2_1(A) ABEA_S4(1, 2, lc, 3, lc, 0, la, A)
#define ABEA_W2_2(A) ABEA_S4(2, 3, lc, 0, ld, 1, la, A)
#define ABEA_W2_3(A) ABEA_S4(3, 0, ld, 1, ld, 2, la, A)
#define ABEA_W3_0(A) ABEA_S4(0, 2, lc, 3, lc, 3, lb, A)
#define ABEA_W3_1(A) ABEA_S4(1, 3, lc, 0, ld, 0, la, A)
#define ABEA_W3_2(A) ABEA_S4(2, 0, ld, 1, ld, 1, la, A)
#define ABEA_W3_3(A) ABEA_S4(3, 1, ld, 2, ld, 2, la, A)
/* the window's registers, event j in the (j mod 5)th: what band B leaves for
 * the next (registers 3 to 0), and where the event after them goes */
#define ABEA_X0 "v5, v6, v7, v11, "
#define ABEA_X1 "v6, v7, v11, v4, "
#define ABEA_X2 "v7, v11, v4, v5, "
#define ABEA_X3 "v11, v4, v5, v6, "
#define ABEA_X4 "v4, v5, v6, v7, "
#define ABEA_B4(Z, S, ST, MV, B, B1, PQ, A, X, RD, XR) \
  "band4%= " #Z ", " #S ", " #B ", " #B1 ", " PQ X #RD ", " #XR ", " ST(A) ", " MV "\n"
#define ABEA_END4(Z, S, ST, B) "end4%= " #Z ", " #S ", " #B ", " ABEA_Q4 ST("q") "\n"
#define ABEA_ROW4_2(Z, S, ST, MV) ABEA_B4(Z, S, ST, MV, 0, 1, ABEA_P4, "p", ABEA_X0, -1, v4) ABEA_END4(Z, S, ST, 1)
#define ABEA_ROW4_4(Z, S, ST, MV)                                                                                 \
  ABEA_B4(Z, S, ST, MV, 0, 1, ABEA_P4, "p", ABEA_X0, 5, v4) ABEA_B4(Z, S, ST, MV, 1, 2, ABEA_Q4, "q", ABEA_X1, 6, v5) \
  ABEA_B4(Z, S, ST, MV, 2, 3, ABEA_P4, "p", ABEA_X2, -1, v6) ABEA_END4(Z, S, ST, 3)
#define ABEA_ROW4_8(Z, S, ST, MV)                                                                                 \
  ABEA_B4(Z, S, ST, MV, 0, 1, ABEA_P4, "p", ABEA_X0, 5, v4) ABEA_B4(Z, S, ST, MV, 1, 2, ABEA_Q4, "q", ABEA_X1, 6, v5) \
  ABEA_B4(Z, S, ST, MV, 2, 3, ABEA_P4, "p", ABEA_X2, 7, v6) ABEA_B4(Z, S, ST, MV, 3, 4, ABEA_Q4, "q", ABEA_X3, 8, v7) \
  ABEA_B4(Z, S, ST, MV, 4, 5, ABEA_P4, "p", ABEA_X4, 9, v11)                                                      \
  ABEA_B4(Z, S, ST, MV, 5, 6, ABEA_Q4, "q", ABEA_X0, 10, v4)                                                      \
  ABEA_B4(Z, S, ST, MV, 6, 7, ABEA_P4, "p", ABEA_X1, -1, v5) ABEA_END4(Z, S, ST, 7)
#define ABEA_WRAP4_2(Z) "wrap4%= " #Z ", 1\n"
#define ABEA_WRAP4_4(Z) ABEA_WRAP4_2(Z) "wrap4%= " #Z ", 2\n wrap4%= " #Z ", 3\n"
#define ABEA_WRAP4_8(Z)                                                                            \
  ABEA_WRAP4_4(Z) "wrap4%= " #Z ", 4\n wrap4%= " #Z ", 5\n wrap4%= " #Z ", 6\n wrap4%= " #Z ", 7\n"
#define ABEA_RUN4(RES, ROW, WRAP, M)                                                                 \
  asm(ABEA_ASM_COMMON "res%==" #RES "\n" ABEA_ASM4 WRAP(0) WRAP(1) ROW(0, 0, M##_0, ".Lb01")                  \
          ROW(0, 1, M##_1, ".Lb02") ROW(0, 2, M##_2, ".Lb03") ROW(0, 3, M##_3, ".Lw0")                          \
          ROW(1, 0, M##_0, ".Lb11") ROW(1, 1, M##_1, ".Lb12") ROW(1, 2, M##_2, ".Lb13")                         \
          ROW(1, 3, M##_3, ".Lw1") ".Lend_%=:\n"                                                               \
      : [p0] "+v"(v.p[0]), [p1] "+v"(v.p[1]), [p2] "+v"(v.p[2]), [p3] "+v"(v.p[3]), [q0] "+v"(v.q[0]),          \
        [q1] "+v"(v.q[1]), [q2] "+v"(v.q[2]), [q3] "+v"(v.q[3]), [td] "+v"(v.td), [tu] "+v"(v.tu),              \
        [lf] "+v"(v.lf), [dg] "+v"(v.dg), [e0] "=&v"(e[0]), [e1] "=&v"(e[1]), [e2] "=&v"(e[2]),                 \
        [e3] "=&v"(e[3]), [t0] "=&v"(t[0]), [t1] "=&v"(t[1]), [t2] "=&v"(t[2]), [t3] "=&v"(t[3]),               \
        [t4] "=&v"(t[4]), [t5] "=&v"(t[5]), [t6] "=&v"(t[6]), [t7] "=&v"(t[7]), [t8] "=&v"(t[8]),               \
        [t9] "=&v"(t[9]), [ta] "=&v"(t[10]), [lo] "=&s"(lo), [cm] "=&s"(cm), [mv] "=&s"(v.mv),                  \
        [K] "+&s"(v.K), [la] "+&s"(la), [lb] "+&s"(lb), [lc] "+&s"(lc), [ld] "+&s"(ld), [le] "+&s"(le)          \
      : [ak] "v"(v.ak), [ax] "v"(v.ax), [calm] "s"(v.calm), [stay] "v"(v.stay), [skip] "v"(v.skip), [step] "v"(v.step) \
      : "v4", "v5", "v6", "v7", "v8", "v9", "v10", "v11", "v12", "v13", "v14", "v16", "v17", "v18", "v20",      \
        "v21", "v22", "vcc", "scc", "memory")
#define ABEA_RUN4_M(RES, ROW, WRAP)                                   \
  if constexpr (M == 0) ABEA_RUN4(RES, ROW, WRAP, ABEA_W0); \
  if constexpr (M == 1) ABEA_RUN4(RES, ROW, WRAP, ABEA_W1); \
  if constexpr (M == 2) ABEA_RUN4(RES, ROW, WRAP, ABEA_W2); \
  if constexpr (M == 3) ABEA_RUN4(RES, ROW, WRAP, ABEA_W3);

/* NB interior bands (2, 4 or 8) at four slots per lane; M = W mod 4; RES the
 * sub-ring of event 0 of the window (1, or 3 in an interval that starts 2 bands
 * after a multiple of 4). */
template <int NB, int M, int RES>
__device__ __forceinline__ void interior(Interior<4> &v, int W) {
  float e[4], t[11];
  uint64_t cm;
  int lo, la = v.K >> 2, lb = la - 1, lc = la + (W >> 2), ld = lc + 1, le = lc - 1;
  static_assert(NB == 2 || NB == 4 || NB == 8, "a refill interval of 2, 4 or 8 bands");
  static_assert(RES == 1 || (RES == 3 && NB == 2), "intervals of 4 or 8 bands start at multiples of 4");
  if constexpr (NB == 8) {
    ABEA_RUN4_M(1, ABEA_ROW4_8, ABEA_WRAP4_8)
  } else if constexpr (NB == 4) {
    ABEA_RUN4_M(1, ABEA_ROW4_4, ABEA_WRAP4_4)
  } else if constexpr (RES == 1) {
    ABEA_RUN4_M(1, ABEA_ROW4_2, ABEA_WRAP4_2)
  } else {
    ABEA_RUN4_M(3, ABEA_ROW4_2, ABEA_WRAP4_2)
  }
}

}  // namespace abea
#endif
