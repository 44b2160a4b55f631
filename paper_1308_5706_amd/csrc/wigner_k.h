// Wigner stage of the directional scale-discretized wavelet transform on gfx950.
//
// Analysis (Sec. 3.2, Eq. 27) for every scale j, m >= 0, m' >= 0 and carried n:
//   U^j_{m m' n} = i^{n-m} sum_l Delta^l_{m'm} Delta^l_{m'n} f_lm conj(Psi^j_ln)
// with Delta = d(pi/2) generated by the three-term recurrence in l on the fly.
// Synthesis (Sec. 3.3, Eq. 34 and Eq. 32 fused) for every l, m >= 0:
//   F_lm = sum_{m' >= 0} Delta^l_{m'm} sum_j kappa^j(l) sum_n sigma_ln Delta^l_{m'n} P^j_{m m' n}(l)
// where P carries the folded quadrature values V of Eq. 35 (computed in stages.hip).
//
// Mapping: a wave owns R consecutive m' ("slots"); its 64 lanes own 64 consecutive
// m.  Each lane runs the l-recurrence of Delta^l_{m'm} for its R pairs, on the rescaled
// values D_l = Delta^l_{m'm} / (g_l(m) h_l(m')) whose Delta^{l-1} coefficient is 1:
//   D_{l+1} = -(ut_l(m') pt_l(m)) D_l - D_{l-1}      (a multiply and an FMA per pair),
// with g_l(m) carried by f_lm (analysis) or applied to the sums (synthesis) and h_l(m') by
// the kappa sigma Delta table.  With alternating signs on D (kernels.h) the recurrence adds the
// product to D_{l-1} in place: a product u p and a multiply-add per pair and step.
//
// The l-range goes in blocks of eight steps, unrolled; the tables and the per-lane arrays are laid
// out by block (kernels.h), so that every address advances by a constant.  About four fifths of the
// vector instructions are FP64 ones, and a multiply-add takes four cycles per SIMD (at two waves per
// SIMD about five were measured), so everything else is kept out of their way.  They do not fill the
// SIMDs: the counters show a vector instruction issued in some 55-65 % of the cycles of the analysis
// and 45-55 % of the synthesis (L = 1024, N = 8 and L = 2048, N = 4); what is left is a wave's own
// chain of steps, with two waves per SIMD to cover it, the barriers, and in the synthesis the window
// sums.
//  * values that depend on (l, m') only -- ut_l(m') and kappa^j(l) sigma_{l,n} Delta^l_{m'n} h_l(m') -- are
//    operands of the multiply-adds through a DPP broadcast (below) instead of scalar loads one step
//    ahead, whose latency the waves waited for;
//  * the analysis reads g_l(m) f_lm and pt_l(m) from LDS, where loads without registers bring the
//    workgroup's rows one or more blocks ahead (once per workgroup, not per wave);
//  * the synthesis sums its window of eight steps over the waves during the next block.
// Measured against the scalar-load form (us, event pairs around the launch): analysis L = 256, N = 8
// 121 -> 48; L = 1024, N = 8 602 -> 396; L = 2048, N = 4 2270 -> 1590.  Synthesis with its final sum:
// 125 -> 91; 738 -> 599; 3360 -> 2580 (there four slots per wave, half the partial sums).
//
// Symmetries used (exact identities of Delta): Delta^l_{m',-n} = (-1)^{l+m'}
// Delta^l_{m'n} lets the l-sum run only over n >= 0 with separate even-l and odd-l
// accumulators; Delta^l_{-m',m} = (-1)^{l+m} Delta^l_{m'm} gives U for m' < 0 from
// m' > 0 (Eq. 29 is then a cosine or sine series).
//
// Extended exponent: the start value Delta^{l0}_{l0,l0} = 2^-l0 is below the double
// range for l0 > 1022, yet the recurrence grows it back to O(1e-2) by l ~ sqrt(2) l0.
// Tiles that hold such start values run the XN variant, which carries each D as
// mantissa * 2^e with e <= 0 and renormalises the mantissa every 8 steps.
#pragma once

#include "s2dw_internal.h"
#include "kernels.h"

#include <type_traits>

namespace s2dw {

namespace {

// z * i^e
__device__ __forceinline__ double2 rot_i(double2 z, int e) {
    e &= 3;
    if (e == 0) return z;
    if (e == 1) return make_double2(-z.y, z.x);
    if (e == 2) return make_double2(-z.x, -z.y);
    return make_double2(z.y, -z.x);
}

constexpr double kBig = 0x1p400;
constexpr double kBigInv = 0x1p-400;

__device__ __forceinline__ double scale_of(int e) { return e < -1074 ? 0.0 : ldexp(1.0, e); }

// A tile (m0, m'0, first segment, first table block) read as wave-uniform values: the addresses
// built from it stay in SGPRs also where the compiler cannot prove that nothing wrote the list.
__device__ __forceinline__ int4 uniform_tile(const int4 *t) {
    const int4 v = *t;
    return make_int4(__builtin_amdgcn_readfirstlane(v.x), __builtin_amdgcn_readfirstlane(v.y),
                     __builtin_amdgcn_readfirstlane(v.z), __builtin_amdgcn_readfirstlane(v.w));
}

// Segment record i (scalar loads).
__device__ __forceinline__ WigSeg seg_of(const WigSeg *segs, int i) {
    typedef const __attribute__((address_space(4))) WigSeg *cptr;
    union {
        WigSeg s;
        int w[sizeof(WigSeg) / 4];
    } v;
    v.s = *(const WigSeg *)(cptr)(segs + i);
#pragma unroll
    for (int k = 0; k < (int)(sizeof(WigSeg) / 4); ++k) v.w[k] = __builtin_amdgcn_readfirstlane(v.w[k]);
    return v.s;
}

// ------------------------------------------------------------- one l-step of one m' slot
// The table values of a step are the same in all lanes.  They sit in VGPRs, 16 consecutive
// values in the 16 lanes of each DPP row (the four rows hold copies), and the FP64 (or FP32)
// multiply-adds read them with row_newbcast: the broadcast costs no instruction, a block of
// eight steps takes K registers per slot however far ahead it is loaded, and vector loads
// return in order, so that the wait for one block leaves the next one in flight (scalar loads
// do not: a wait for one waits for all).  The steps are written as one asm statement each:
// the DPP form of the FP64 multiply-add is not selected from a broadcast and an fma.  A VALU write
// of a register needs two wait states before a DPP read of it; each statement opens with
// instructions that read no table value, so that a copy placed before it stays apart.
// Entry i of the step is table value FLAT + i of the block: register (FLAT + i) / 16, lane
// (FLAT + i) % 16 of the row.

#define S2DW_DPP(LN) " row_newbcast:%[" LN "] row_mask:0xf bank_mask:0xf\n\t"

// the recurrence: F0 += (u p) F1, the product u p rounded as the unsigned form has it
#define S2DW_REC                              \
    "v_mov_b64_dpp %[w], %[u]" S2DW_DPP("lu") \
    "v_mul_f64 %[w], %[w], %[p]\n\t"          \
    "v_fmac_f64_e32 %[F0], %[w], %[F1]\n\t"
// analysis: acc[i] += kb_i (x f)
#define S2DW_WE(i) "v_fmac_f64_dpp %[a" #i "], %[t" #i "], %[gr]" S2DW_DPP("l" #i) \
                   "v_fmac_f64_dpp %[b" #i "], %[t" #i "], %[gi]" S2DW_DPP("l" #i)
#define S2DW_WO(i) [a##i] "+v"(A[E0 + i][0]), [b##i] "+v"(A[E0 + i][1])
#define S2DW_WI(i) [t##i] "v"(tab[(FLAT + E0 + i) / 16]), [l##i] "n"((FLAT + E0 + i) % 16)
#define S2DW_WHEAD                      \
    "v_mul_f64 %[gr], %[fx], %[x]\n\t"  \
    "v_mul_f64 %[gi], %[fy], %[x]\n\t"  \
    S2DW_REC
#define S2DW_WHEAD_O [w] "=&v"(w), [gr] "=&v"(gr), [gi] "=&v"(gi), [F0] "+v"(F0)
#define S2DW_WHEAD_I [F1] "v"(F1), [x] "v"(x), [fx] "v"(f.x), [fy] "v"(f.y), [p] "v"(p), [u] "v"(u), [lu] "n"(S)

// the entries E0 .. E0 + NE - 1 alone (K > 4: the entries of one scale slot)
template <int NE, int E0, int FLAT, int NT, int NA>
__device__ __forceinline__ void wig_fwd_tail(double (&A)[NA][2], const double (&tab)[NT], double gr, double gi) {
    if constexpr (NE == 5)
        asm volatile("s_nop 1\n\t" S2DW_WE(0) S2DW_WE(1) S2DW_WE(2) S2DW_WE(3) S2DW_WE(4)
            : S2DW_WO(0), S2DW_WO(1), S2DW_WO(2), S2DW_WO(3), S2DW_WO(4)
            : S2DW_WI(0), S2DW_WI(1), S2DW_WI(2), S2DW_WI(3), S2DW_WI(4), [gr] "v"(gr), [gi] "v"(gi));
    else if constexpr (NE == 6)
        asm volatile("s_nop 1\n\t" S2DW_WE(0) S2DW_WE(1) S2DW_WE(2) S2DW_WE(3) S2DW_WE(4) S2DW_WE(5)
            : S2DW_WO(0), S2DW_WO(1), S2DW_WO(2), S2DW_WO(3), S2DW_WO(4), S2DW_WO(5)
            : S2DW_WI(0), S2DW_WI(1), S2DW_WI(2), S2DW_WI(3), S2DW_WI(4), S2DW_WI(5), [gr] "v"(gr), [gi] "v"(gi));
    else if constexpr (NE == 7)
        asm volatile("s_nop 1\n\t" S2DW_WE(0) S2DW_WE(1) S2DW_WE(2) S2DW_WE(3) S2DW_WE(4) S2DW_WE(5) S2DW_WE(6)
            : S2DW_WO(0), S2DW_WO(1), S2DW_WO(2), S2DW_WO(3), S2DW_WO(4), S2DW_WO(5), S2DW_WO(6)
            : S2DW_WI(0), S2DW_WI(1), S2DW_WI(2), S2DW_WI(3), S2DW_WI(4), S2DW_WI(5), S2DW_WI(6), [gr] "v"(gr),
              [gi] "v"(gi));
    else
        asm volatile("s_nop 1\n\t" S2DW_WE(0) S2DW_WE(1) S2DW_WE(2) S2DW_WE(3) S2DW_WE(4) S2DW_WE(5) S2DW_WE(6) S2DW_WE(7)
            : S2DW_WO(0), S2DW_WO(1), S2DW_WO(2), S2DW_WO(3), S2DW_WO(4), S2DW_WO(5), S2DW_WO(6), S2DW_WO(7)
            : S2DW_WI(0), S2DW_WI(1), S2DW_WI(2), S2DW_WI(3), S2DW_WI(4), S2DW_WI(5), S2DW_WI(6), S2DW_WI(7),
              [gr] "v"(gr), [gi] "v"(gi));
}

// Step S (0..7) of a block: F1 = D_l (x: its value, F1 itself without the extended exponent), F0 =
// D_{l-1} on entry and D_{l+1} on exit (with the signs of the rescaled recurrence, see above).
template <int K, int S>
__device__ __forceinline__ void wig_fwd_step(double (&A)[2 * K][2], double &F0, double F1, double x, double2 f,
                                             double p, double u, const double (&tab)[K]) {
    constexpr int FLAT = S * 2 * K, E0 = 0;
    double w, gr, gi;
    if constexpr (K == 1) {
        asm volatile(S2DW_WHEAD S2DW_WE(0) S2DW_WE(1)
            : S2DW_WHEAD_O, S2DW_WO(0), S2DW_WO(1)
            : S2DW_WHEAD_I, S2DW_WI(0), S2DW_WI(1));
    } else if constexpr (K == 2) {
        asm volatile(S2DW_WHEAD S2DW_WE(0) S2DW_WE(1) S2DW_WE(2) S2DW_WE(3)
            : S2DW_WHEAD_O, S2DW_WO(0), S2DW_WO(1), S2DW_WO(2), S2DW_WO(3)
            : S2DW_WHEAD_I, S2DW_WI(0), S2DW_WI(1), S2DW_WI(2), S2DW_WI(3));
    } else if constexpr (K == 3) {
        asm volatile(S2DW_WHEAD S2DW_WE(0) S2DW_WE(1) S2DW_WE(2) S2DW_WE(3) S2DW_WE(4) S2DW_WE(5)
            : S2DW_WHEAD_O, S2DW_WO(0), S2DW_WO(1), S2DW_WO(2), S2DW_WO(3), S2DW_WO(4), S2DW_WO(5)
            : S2DW_WHEAD_I, S2DW_WI(0), S2DW_WI(1), S2DW_WI(2), S2DW_WI(3), S2DW_WI(4), S2DW_WI(5));
    } else if constexpr (K == 4) {
        asm volatile(S2DW_WHEAD S2DW_WE(0) S2DW_WE(1) S2DW_WE(2) S2DW_WE(3) S2DW_WE(4) S2DW_WE(5) S2DW_WE(6) S2DW_WE(7)
            : S2DW_WHEAD_O, S2DW_WO(0), S2DW_WO(1), S2DW_WO(2), S2DW_WO(3), S2DW_WO(4), S2DW_WO(5), S2DW_WO(6),
              S2DW_WO(7)
            : S2DW_WHEAD_I, S2DW_WI(0), S2DW_WI(1), S2DW_WI(2), S2DW_WI(3), S2DW_WI(4), S2DW_WI(5), S2DW_WI(6),
              S2DW_WI(7));
    } else {
        asm volatile(S2DW_WHEAD : S2DW_WHEAD_O : S2DW_WHEAD_I);
        wig_fwd_tail<K, 0, FLAT>(A, tab, gr, gi);
        wig_fwd_tail<K, K, FLAT>(A, tab, gr, gi);
    }
}

// synthesis: y = sum_i kb_i v_i, (fr, fi) += x y.  FP64: double table and sums.
#define S2DW_YE(i) "v_fmac_f64_dpp %[yr], %[t" #i "], %[a" #i "]" S2DW_DPP("l" #i) \
                   "v_fmac_f64_dpp %[yi], %[t" #i "], %[b" #i "]" S2DW_DPP("l" #i)
#define S2DW_YF(i) "v_fmac_f32_dpp %[yr], %[t" #i "], %[a" #i "]" S2DW_DPP("l" #i) \
                   "v_fmac_f32_dpp %[yi], %[t" #i "], %[b" #i "]" S2DW_DPP("l" #i)
#define S2DW_YI(i) [t##i] "v"(tab[(FLAT + E0 + i) / 16]), [l##i] "n"((FLAT + E0 + i) % 16), [a##i] "v"(V[E0 + i][0]), \
                   [b##i] "v"(V[E0 + i][1])
#define S2DW_AREC "s_nop 1\n\t" S2DW_REC
#define S2DW_AFIRST                                           \
    "v_mov_b64_dpp %[c], %[t0]" S2DW_DPP("l0")                \
    "v_mul_f64 %[yr], %[c], %[a0]\n\t"                        \
    "v_mul_f64 %[yi], %[c], %[b0]\n\t"
#define S2DW_AFIRSTF                                          \
    "v_mul_f32_dpp %[yr], %[t0], %[a0]" S2DW_DPP("l0")        \
    "v_mul_f32_dpp %[yi], %[t0], %[b0]" S2DW_DPP("l0")
#define S2DW_ALAST "v_fmac_f64_e32 %[fr], %[x], %[yr]\n\tv_fmac_f64_e32 %[fi], %[x], %[yi]\n\t"
#define S2DW_ALASTF "v_fmac_f32_e32 %[fr], %[x], %[yr]\n\tv_fmac_f32_e32 %[fi], %[x], %[yi]\n\t"
#define S2DW_AREC_O [w] "=&v"(w), [F0] "+v"(F0)
#define S2DW_AREC_I [F1] "v"(F1), [p] "v"(p), [u] "v"(u), [lu] "n"(S)

// the sums of NE entries from E0 (K > 4: one scale slot at a time)
template <int NE, int E0, int FLAT, int NT, int NA>
__device__ __forceinline__ void wig_adj_sum(const double (&V)[NA][2], const double (&tab)[NT], double x, double &fr,
                                            double &fi) {
    double c, yr, yi;
#define S2DW_ASUM(ENTS, INS)                                                                                         \
    asm volatile("s_nop 1\n\t" S2DW_AFIRST ENTS S2DW_ALAST                                                                  \
        : [c] "=&v"(c), [yr] "=&v"(yr), [yi] "=&v"(yi), [fr] "+v"(fr), [fi] "+v"(fi)                                \
        : [x] "v"(x), S2DW_YI(0) INS)
#define S2DW_C ,
    if constexpr (NE == 5)
        S2DW_ASUM(S2DW_YE(1) S2DW_YE(2) S2DW_YE(3) S2DW_YE(4),
                  S2DW_C S2DW_YI(1) S2DW_C S2DW_YI(2) S2DW_C S2DW_YI(3) S2DW_C S2DW_YI(4));
    else if constexpr (NE == 6)
        S2DW_ASUM(S2DW_YE(1) S2DW_YE(2) S2DW_YE(3) S2DW_YE(4) S2DW_YE(5),
                  S2DW_C S2DW_YI(1) S2DW_C S2DW_YI(2) S2DW_C S2DW_YI(3) S2DW_C S2DW_YI(4) S2DW_C S2DW_YI(5));
    else if constexpr (NE == 7)
        S2DW_ASUM(S2DW_YE(1) S2DW_YE(2) S2DW_YE(3) S2DW_YE(4) S2DW_YE(5) S2DW_YE(6),
                  S2DW_C S2DW_YI(1) S2DW_C S2DW_YI(2) S2DW_C S2DW_YI(3) S2DW_C S2DW_YI(4) S2DW_C S2DW_YI(5)
                      S2DW_C S2DW_YI(6));
    else
        S2DW_ASUM(S2DW_YE(1) S2DW_YE(2) S2DW_YE(3) S2DW_YE(4) S2DW_YE(5) S2DW_YE(6) S2DW_YE(7),
                  S2DW_C S2DW_YI(1) S2DW_C S2DW_YI(2) S2DW_C S2DW_YI(3) S2DW_C S2DW_YI(4) S2DW_C S2DW_YI(5)
                      S2DW_C S2DW_YI(6) S2DW_C S2DW_YI(7));
#undef S2DW_ASUM
}
template <int NE, int E0, int FLAT, int NT, int NA>
__device__ __forceinline__ void wig_adj_sum(const float (&V)[NA][2], const float (&tab)[NT], float x, float &fr,
                                            float &fi) {
    float yr, yi;
#define S2DW_ASUM(ENTS, INS)                                                                                         \
    asm volatile("s_nop 1\n\t" S2DW_AFIRSTF ENTS S2DW_ALASTF                                                                \
        : [yr] "=&v"(yr), [yi] "=&v"(yi), [fr] "+v"(fr), [fi] "+v"(fi)                                              \
        : [x] "v"(x), S2DW_YI(0) INS)
    if constexpr (NE == 5)
        S2DW_ASUM(S2DW_YF(1) S2DW_YF(2) S2DW_YF(3) S2DW_YF(4),
                  S2DW_C S2DW_YI(1) S2DW_C S2DW_YI(2) S2DW_C S2DW_YI(3) S2DW_C S2DW_YI(4));
    else if constexpr (NE == 6)
        S2DW_ASUM(S2DW_YF(1) S2DW_YF(2) S2DW_YF(3) S2DW_YF(4) S2DW_YF(5),
                  S2DW_C S2DW_YI(1) S2DW_C S2DW_YI(2) S2DW_C S2DW_YI(3) S2DW_C S2DW_YI(4) S2DW_C S2DW_YI(5));
    else if constexpr (NE == 7)
        S2DW_ASUM(S2DW_YF(1) S2DW_YF(2) S2DW_YF(3) S2DW_YF(4) S2DW_YF(5) S2DW_YF(6),
                  S2DW_C S2DW_YI(1) S2DW_C S2DW_YI(2) S2DW_C S2DW_YI(3) S2DW_C S2DW_YI(4) S2DW_C S2DW_YI(5)
                      S2DW_C S2DW_YI(6));
    else
        S2DW_ASUM(S2DW_YF(1) S2DW_YF(2) S2DW_YF(3) S2DW_YF(4) S2DW_YF(5) S2DW_YF(6) S2DW_YF(7),
                  S2DW_C S2DW_YI(1) S2DW_C S2DW_YI(2) S2DW_C S2DW_YI(3) S2DW_C S2DW_YI(4) S2DW_C S2DW_YI(5)
                      S2DW_C S2DW_YI(6) S2DW_C S2DW_YI(7));
#undef S2DW_ASUM
}

template <int K, int S>
__device__ __forceinline__ void wig_adj_step(const double (&V)[2 * K][2], double &F0, double F1, double x, double p,
                                             double u, const double (&tab)[K], double &fr, double &fi) {
    constexpr int FLAT = S * 2 * K, E0 = 0;
    double w, c, yr, yi;
#define S2DW_ASTEP(ENTS, INS)                                                                                        \
    asm volatile(S2DW_AREC S2DW_AFIRST ENTS S2DW_ALAST                                                                      \
        : S2DW_AREC_O, [c] "=&v"(c), [yr] "=&v"(yr), [yi] "=&v"(yi), [fr] "+v"(fr), [fi] "+v"(fi)                   \
        : S2DW_AREC_I, [x] "v"(x), S2DW_YI(0) INS)
    if constexpr (K == 1) S2DW_ASTEP(S2DW_YE(1), S2DW_C S2DW_YI(1));
    else if constexpr (K == 2)
        S2DW_ASTEP(S2DW_YE(1) S2DW_YE(2) S2DW_YE(3), S2DW_C S2DW_YI(1) S2DW_C S2DW_YI(2) S2DW_C S2DW_YI(3));
    else if constexpr (K == 3)
        S2DW_ASTEP(S2DW_YE(1) S2DW_YE(2) S2DW_YE(3) S2DW_YE(4) S2DW_YE(5),
                   S2DW_C S2DW_YI(1) S2DW_C S2DW_YI(2) S2DW_C S2DW_YI(3) S2DW_C S2DW_YI(4) S2DW_C S2DW_YI(5));
    else if constexpr (K == 4)
        S2DW_ASTEP(S2DW_YE(1) S2DW_YE(2) S2DW_YE(3) S2DW_YE(4) S2DW_YE(5) S2DW_YE(6) S2DW_YE(7),
                   S2DW_C S2DW_YI(1) S2DW_C S2DW_YI(2) S2DW_C S2DW_YI(3) S2DW_C S2DW_YI(4) S2DW_C S2DW_YI(5)
                       S2DW_C S2DW_YI(6) S2DW_C S2DW_YI(7));
    else {
        asm volatile(S2DW_AREC : S2DW_AREC_O : S2DW_AREC_I);
        wig_adj_sum<K, 0, FLAT>(V, tab, x, fr, fi);
        wig_adj_sum<K, K, FLAT>(V, tab, x, fr, fi);
    }
#undef S2DW_ASTEP
}
template <int K, int S>
__device__ __forceinline__ void wig_adj_step(const float (&V)[2 * K][2], double &F0, double F1, float x, double p,
                                             double u, const float (&tab)[K], float &fr, float &fi) {
    constexpr int FLAT = S * 2 * K, E0 = 0;
    double w;
    float yr, yi;
#define S2DW_ASTEP(ENTS, INS)                                                                                        \
    asm volatile(S2DW_AREC S2DW_AFIRSTF ENTS S2DW_ALASTF                                                                    \
        : S2DW_AREC_O, [yr] "=&v"(yr), [yi] "=&v"(yi), [fr] "+v"(fr), [fi] "+v"(fi)                                 \
        : S2DW_AREC_I, [x] "v"(x), S2DW_YI(0) INS)
    if constexpr (K == 1) S2DW_ASTEP(S2DW_YF(1), S2DW_C S2DW_YI(1));
    else if constexpr (K == 2)
        S2DW_ASTEP(S2DW_YF(1) S2DW_YF(2) S2DW_YF(3), S2DW_C S2DW_YI(1) S2DW_C S2DW_YI(2) S2DW_C S2DW_YI(3));
    else if constexpr (K == 3)
        S2DW_ASTEP(S2DW_YF(1) S2DW_YF(2) S2DW_YF(3) S2DW_YF(4) S2DW_YF(5),
                   S2DW_C S2DW_YI(1) S2DW_C S2DW_YI(2) S2DW_C S2DW_YI(3) S2DW_C S2DW_YI(4) S2DW_C S2DW_YI(5));
    else if constexpr (K == 4)
        S2DW_ASTEP(S2DW_YF(1) S2DW_YF(2) S2DW_YF(3) S2DW_YF(4) S2DW_YF(5) S2DW_YF(6) S2DW_YF(7),
                   S2DW_C S2DW_YI(1) S2DW_C S2DW_YI(2) S2DW_C S2DW_YI(3) S2DW_C S2DW_YI(4) S2DW_C S2DW_YI(5)
                       S2DW_C S2DW_YI(6) S2DW_C S2DW_YI(7));
    else {
        asm volatile(S2DW_AREC : S2DW_AREC_O : S2DW_AREC_I);
        wig_adj_sum<K, 0, FLAT>(V, tab, x, fr, fi);
        wig_adj_sum<K, K, FLAT>(V, tab, x, fr, fi);
    }
#undef S2DW_ASTEP
}
#undef S2DW_C

// The table value of a step after which register q of a block of K registers is free: its last
// use is step (16 q + 15) / 2K.
constexpr int tab_last(int K, int q) { return (16 * q + 15) / (2 * K); }

// Loads through a buffer descriptor: a uniform byte offset (an SGPR, advanced by one scalar addition)
// and a 32-bit lane offset, so that a load ahead costs neither address registers nor vector
// instructions.  All offsets stay within the arrays (below 2^32 bytes), which carry the rows that
// are read ahead.
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_of(const void *p) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, 0xffffffffu, 0x00027000);
}
__device__ __forceinline__ double buf_f64(__amdgpu_buffer_rsrc_t b, unsigned lane_off, unsigned off) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(b, lane_off, off, 0));
}
__device__ __forceinline__ u32x4 buf_b128(__amdgpu_buffer_rsrc_t b, unsigned lane_off, unsigned off) {
    return __builtin_amdgcn_raw_buffer_load_b128(b, lane_off, off, 0);
}
// The same descriptor as plain words, for the loads that go straight to LDS: 16 bytes per active
// lane, lane i to LDS byte lds + 16 i.  They return in order; wait_lds<N> waits until at most N
// vector memory operations are in flight.  (Written out because the compiler would wait for all
// of them before the next read of LDS; its own waits count its own operations only, and with
// these in flight beside them they wait for more, not less.)  A scalar register that a vector
// instruction wrote (a readfirstlane of off, of the descriptor) is not read by a vector memory
// instruction within five wait states; the compiler keeps that distance for its own loads but not
// into a statement, which therefore keeps it itself: the move to m0 and four more.
__device__ __forceinline__ u32x4 desc_of(const void *p) {
    const unsigned long long v = (unsigned long long)p;
    u32x4 d;
    d.x = __builtin_amdgcn_readfirstlane((unsigned)v);
    d.y = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32) & 0xffffu);
    d.z = 0xffffffffu;
    d.w = 0x00027000u;
    return d;
}
// One of these loads, after the move to m0 and WAIT + 1 wait states.
#define S2DW_LDS_LOAD(D, LANE, OFF, LDS, WAIT) \
    "s_mov_b32 m0, %[" LDS "]\n\ts_nop " WAIT "\n\tbuffer_load_dwordx4 %[" LANE "], %[" D "], %[" OFF "] offen lds\n\t"
// The lanes below 64 - %[N] only.
#define S2DW_LDS_LANES(N) "s_lshr_b64 exec, -1, %[" N "]\n\t"

// What a load takes beside the lane offset.
struct LdsLoad {
    u32x4 d;
    unsigned off, lds;
};
__device__ __forceinline__ LdsLoad lds_load(u32x4 d, unsigned off, unsigned lds) {
    return {d, (unsigned)__builtin_amdgcn_readfirstlane(off), (unsigned)__builtin_amdgcn_readfirstlane(lds)};
}
// The five loads of a block in one statement, with the wait states of one: a, the same lanes at off_a2
// to lds_a2, b, and c and d by the first NC and ND lanes.  Every lane is active where it stands.
template <int NC, int ND>
__device__ __forceinline__ void load_lds16_5(const LdsLoad &a, unsigned lane_a, unsigned off_a2, unsigned lds_a2,
                                             const LdsLoad &b, unsigned lane_b, const LdsLoad &c, unsigned lane_c,
                                             const LdsLoad &d, unsigned lane_d) {
    static_assert(NC > 0 && NC <= 64 && ND > 0 && ND <= 64, "lanes");
    unsigned long long exec;
    asm volatile(S2DW_LDS_LOAD("da", "va", "oa", "la", "3") S2DW_LDS_LOAD("da", "va", "oa2", "la2", "0")
                     S2DW_LDS_LOAD("db", "vb", "ob", "lb", "0") "s_mov_b64 %[ex], exec\n\t" S2DW_LDS_LANES("nc")
                         S2DW_LDS_LOAD("dc", "vc", "oc", "lc", "0") S2DW_LDS_LANES("nd")
                             S2DW_LDS_LOAD("dd", "vd", "od", "ld", "0") "s_mov_b64 exec, %[ex]"
                 : [ex] "=&s"(exec)
                 : [da] "s"(a.d), [oa] "s"(a.off), [la] "s"(a.lds), [va] "v"(lane_a),
                   [oa2] "s"(__builtin_amdgcn_readfirstlane(off_a2)), [la2] "s"(__builtin_amdgcn_readfirstlane(lds_a2)),
                   [db] "s"(b.d), [ob] "s"(b.off), [lb] "s"(b.lds), [vb] "v"(lane_b), [dc] "s"(c.d), [oc] "s"(c.off),
                   [lc] "s"(c.lds), [vc] "v"(lane_c), [dd] "s"(d.d), [od] "s"(d.off), [ld] "s"(d.lds), [vd] "v"(lane_d),
                   [nc] "n"(64 - NC), [nd] "n"(64 - ND)
                 : "m0", "scc", "memory");
}
#undef S2DW_LDS_LANES
#undef S2DW_LDS_LOAD
template <int N>
__device__ __forceinline__ void wait_lds() {
    static_assert(N >= 0 && N < 64, "vmcnt");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ unsigned lds_off(const void *p) {
    return __builtin_amdgcn_readfirstlane((unsigned)(unsigned long long)p);
}
// A workgroup barrier for LDS traffic alone: loads and stores to memory stay in flight.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Unrolls f(integral_constant<0>) .. f(integral_constant<7>).
template <class F>
__device__ __forceinline__ void eight(F f) {
    f(std::integral_constant<int, 0>());
    f(std::integral_constant<int, 1>());
    f(std::integral_constant<int, 2>());
    f(std::integral_constant<int, 3>());
    f(std::integral_constant<int, 4>());
    f(std::integral_constant<int, 5>());
    f(std::integral_constant<int, 6>());
    f(std::integral_constant<int, 7>());
}

// The table values of a wave's R slots pass through LDS, NS blocks of them: brought there once each,
// in 16-byte pieces, and read from there in the replicated form the DPP reads need.  (Loaded in
// that form straight from memory, each register cost the vector cache as many accesses as four
// ordinary loads, and it was the limit.)  The slots belong to one wave.
template <int K, int R, typename T, int NS>
struct alignas(16) WigSlots {
    T tab[NS][R][16 * K];
    double u[NS][R][8];
};

// The state of a wave's R recurrences.
template <int R>
struct alignas(16) WigState {
    double F0[R][64], F1[R][64];
    int ex[R][64];
};

// The l-recurrence of a wave's R slots with the table values of its block, shared by both
// directions.  T: type of the table (double, or float in the mixed synthesis).
template <int K, int R, bool XN, typename T, int NS>
struct WigRows {
    double F0[R], F1[R];      // D_{l-1}, D_l at the start of a block
    double scl[R];            // extended exponent: D = F scl
    int ex[R];
    int l0[R];                // first l of the lane and slot
    double sv[R];             // value there (mantissa with the extended exponent)
    int se[R];
    T tab[R][K];              // the block's table values
    double u[R], un[R];       // u of the block and of the next one
    T tn[R];                  // K = 1: the next block's table values (else they roll)
    WigSlots<K, R, T, NS> *sl;
    int lane16, lane;
    unsigned to, uo;          // byte offsets of the 16 bytes of table and u values that the lane brings
    int mp0;                  // row of the wave's first slot

    static constexpr int kTabLanes = R * 16 * K * (int)sizeof(T) / 16;  // lanes that bring table values
    static constexpr int kULanes = R * 4;                               // and u values
    static_assert(kTabLanes <= 64 && kULanes <= 64, "one load per block");

    __device__ __forceinline__ void init(const double *seed, const double *seedm, const int *seede, int L, int Lp,
                                         int kstride, int ustride, int m, int mpb, int lane_,
                                         WigSlots<K, R, T, NS> *slots) {
        lane = lane_;
        lane16 = lane & 15;
        sl = slots;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int mpv = mpb + r;
            const int mp = mpv < L ? mpv : L - 1;
            l0[r] = max(m, mpv);
            const bool ok = mpv < L && m < L;
            const size_t si = (size_t)mp * Lp + (m < Lp ? m : Lp - 1);
            if (XN) {
                sv[r] = ok ? seedm[si] : 0.0;
                se[r] = ok ? seede[si] : 0;
            } else {
                sv[r] = ok ? seed[si] : 0.0;
                se[r] = 0;
            }
            F0[r] = F1[r] = 0.0;
            ex[r] = 0;
            scl[r] = 1.0;
        }
        mp0 = mpb < L ? mpb : L - 1;
        const int rmax = L - 1 - mp0;  // slots beyond L take the row L - 1
        constexpr int per = kTabLanes / R;
        const int tr = min(min(lane / per, R - 1), rmax), ur = min(min(lane >> 2, R - 1), rmax);
        to = (unsigned)(tr * kstride) * (unsigned)sizeof(T) + (unsigned)(lane % per) * 16u;
        uo = (unsigned)(ur * ustride) * (unsigned)sizeof(double) + (unsigned)(lane & 3) * 16u;
    }
    __device__ __forceinline__ T get(int s, int r, int q) const { return sl->tab[s][r][q * 16 + lane16]; }
    __device__ __forceinline__ double getu(int s, int r) const { return sl->u[s][r][lane & 7]; }
    // the values of the first block (in LDS slot s)
    __device__ __forceinline__ void first(int s) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
#pragma unroll
            for (int q = 0; q < K; ++q) tab[r][q] = get(s, r, q);
            u[r] = getu(s, r);
        }
    }
    // after step S: the registers it used last take the next block's values (LDS slot s), from
    // step FROM on
    template <int S, int FROM>
    __device__ __forceinline__ void roll(int s) {
        if constexpr (S == 5) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                un[r] = getu(s, r);
                if constexpr (K == 1) tn[r] = get(s, r, 0);
            }
        }
        if constexpr (K > 1) {
#pragma unroll
            for (int q = 0; q < K; ++q)
                if ((tab_last(K, q) > FROM ? tab_last(K, q) : FROM) == S) {
#pragma unroll
                    for (int r = 0; r < R; ++r) tab[r][q] = get(s, r, q);
                }
        }
    }
    __device__ __forceinline__ void advance() {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            u[r] = un[r];
            if constexpr (K == 1) tab[r][0] = tn[r];
        }
    }
    // the start values of the lanes that begin at l
    template <int S>
    __device__ __forceinline__ void start(int l) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            double &c = (S & 1) ? F0[r] : F1[r];
            const bool h = l == l0[r];
            c = h ? sv[r] : c;
            if (XN) {
                ex[r] = h ? se[r] : ex[r];
                if (h) scl[r] = scale_of(se[r]);
            }
        }
    }
    __device__ __forceinline__ void renorm() {
        if (!XN) return;
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (fabs(F1[r]) > kBig) {
                F1[r] *= kBigInv;
                F0[r] *= kBigInv;
                ex[r] += 400;
                scl[r] = scale_of(ex[r]);
            }
    }
    // The state at the start of a block that is taken twice, kept in LDS (the wave's own).
    __device__ __forceinline__ void save(WigState<R> *b) const {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            b->F0[r][lane] = F0[r];
            b->F1[r][lane] = F1[r];
            if (XN) b->ex[r][lane] = ex[r];
        }
    }
    __device__ __forceinline__ void restore(const WigState<R> *b) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            F0[r] = b->F0[r][lane];
            F1[r] = b->F1[r][lane];
            if (XN) {
                ex[r] = b->ex[r][lane];
                scl[r] = scale_of(ex[r]);
            }
        }
    }
};

}  // namespace

// ------------------------------------------------------------------------------- analysis

// Table blocks of the analysis kernel's values held in LDS: the one in use, the next, and those on
// their way.  A block is requested NS - 2 blocks before it is needed; measured at L = 1024, N = 8,
// a load takes about a block of two resident waves per SIMD, and with one slot and order per
// wave (small L: few waves, short blocks) several.  No more of them than let two workgroups share a
// CU's LDS: with six blocks for one slot one was left, and launches of more workgroups than CUs
// waited (us, six against five: 64 maps of L = 48, N = 4 35 against 27; one map of L = 421, N = 6 62
// against 49; of L = 256, N = 8 39 with either).
template <int K, int R>
constexpr int wig_fwd_slots() { return K >= 5 ? 4 : (R == 1 ? 5 : (R == 2 ? 4 : 3)); }

template <int K, int R>
struct alignas(16) WigFwdLds {
    static constexpr int NS = wig_fwd_slots<K, R>();
    double2 f[NS][8][64];                  // g f_lm of the workgroup's 64 m, by step
    double p[NS][8][64];                   // pt
    WigSlots<K, R, double, NS> s[4];
    WigState<R> saved[4];
};

// Tile bx of map by; thread tid of 256.
template <int K, int R, bool XN>
__device__ __forceinline__ void wig_fwd_body(const WigFwdArgs &a, WigFwdLds<K, R> *lds, int bx, int by, int tid) {
    constexpr int NS = WigFwdLds<K, R>::NS;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
    const int4 t = uniform_tile(a.tiles + bx);
    const int L = a.L, Lp = a.Lp;
    const int m = t.x + lane;
    const int mpb = t.y + wave * R;                                // slots beyond L run along, unused
    const int lhead = min(L - 1, max(t.x + 63, t.y + 4 * R - 1));  // every lane of the workgroup has started

    WigRows<K, R, XN, double, NS> w;
    w.init(a.seed, a.seedm, a.seede, L, Lp, a.kstride, a.ustride, m, mpb, lane, &lds->s[wave]);
    // acc[r][l parity][scale slot, k][re, im]
    double acc[R][2][2 * K][2];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int i = 0; i < 2 * K; ++i) acc[r][p][i][0] = acc[r][p][i][1] = 0.0;

    // The per-lane values go by row: row 8 blk + S is step S of table block blk (f is zero there
    // for an l outside the segment).  Wave w brings the rows 2w and 2w + 1 of a block for the
    // workgroup, and its own slots' table and u values.
    const u32x4 fd = desc_of(a.fpad + by * a.s_fpad), pd = desc_of(a.pq);
    const u32x4 td = desc_of(a.kb2 + (size_t)w.mp0 * a.kstride), ud = desc_of(a.uv + (size_t)w.mp0 * a.ustride);
    const unsigned fo = (unsigned)m * 16u;
    const unsigned po = (unsigned)(lane >> 5) * ((unsigned)Lp * 8u) + (unsigned)t.x * 8u + (unsigned)(lane & 31) * 16u;
    const unsigned lf = lds_off(&lds->f[0][2 * wave][0]), lp = lds_off(&lds->p[0][2 * wave][0]);
    const unsigned lt = lds_off(&lds->s[wave].tab[0][0][0]), lu = lds_off(&lds->s[wave].u[0][0][0]);
    constexpr int kLoads = 5;  // per wave and block
    auto request = [&](int blk, int slot) {
        const unsigned row = (unsigned)blk * 8u + 2u * (unsigned)wave, ro = row * (unsigned)Lp * 8u;
        load_lds16_5<decltype(w)::kTabLanes, decltype(w)::kULanes>(
            lds_load(fd, 2u * ro, lf + (unsigned)slot * 8192u), fo, 2u * ro + (unsigned)Lp * 16u,
            lf + (unsigned)slot * 8192u + 1024u, lds_load(pd, ro, lp + (unsigned)slot * 4096u), po,
            lds_load(td, (unsigned)blk * (128u * K), lt + (unsigned)slot * (R * K * 128u)), w.to,
            lds_load(ud, (unsigned)blk * 64u, lu + (unsigned)slot * (R * 64u)), w.uo);
    };

    int si = t.z, blk = t.w;
    WigSeg sg = seg_of(a.segs, si), sgn = seg_of(a.segs, si + 1);
    int lo = max(sg.s0, max(t.x, t.y));
    int lb = lo & ~7;
    int cur = 0;                        // LDS slot of the block
    double2 f[2];
    double p[2];
    auto load_f = [&](int i, int slot, int S) {
        f[i] = lds->f[slot][S][lane];
        p[i] = lds->p[slot][S][lane];
    };

    // The block of steps lb .. lb + 7 (table block blk); returns whether it ends the segment, and
    // moves on to the next block: the same steps again where the segment ends inside it, from
    // the state at its start.  HEAD: some lane starts in it; then only the segment's steps are
    // run, and a block that is taken again goes on from where it was left (the first segments
    // are short: at L = 64 the eight steps from l = 0 belong to four of them).
    auto block = [&](auto head_c) {
        constexpr bool HEAD = decltype(head_c)::value;
        const bool last = lb + 8 >= sg.s1;
        const int nxt = cur + 1 < NS ? cur + 1 : 0;
        if (!HEAD && last && (sg.s1 & 7)) w.save(&lds->saved[wave]);
        eight([&](auto s_c) {
            constexpr int S = decltype(s_c)::value;
            if constexpr (S < 7) load_f((S + 1) & 1, cur, S + 1);
            else load_f(0, nxt, 0);
            if constexpr (S == 4) {
                // the next block has arrived in every wave, and every wave has left the last one:
                // its LDS slot takes the block NS - 1 ahead
                wait_lds<kLoads * (NS - 3)>();
                lds_barrier();
                request(blk + NS - 1, cur > 0 ? cur - 1 : NS - 1);
            }
            if (!HEAD || (lb + S >= lo && lb + S < sg.s1)) {
                if constexpr (HEAD) w.template start<S>(lb + S);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    double &F0 = (S & 1) ? w.F1[r] : w.F0[r];
                    const double F1 = (S & 1) ? w.F0[r] : w.F1[r];
                    const double x = XN ? F1 * w.scl[r] : F1;
                    wig_fwd_step<K, S>(acc[r][S & 1], F0, F1, x, f[S & 1], p[S & 1], w.u[r], w.tab[r]);
                }
            }
            w.template roll<S, 4>(nxt);
            __builtin_amdgcn_sched_barrier(0);
        });
        if (!HEAD || !last || !(sg.s1 & 7)) w.renorm();
        w.advance();
        ++blk;
        cur = nxt;
        lb = last ? sg.s1 & ~7 : lb + 8;
        return last;
    };

    auto flush = [&](int slot, int Lj, long long off) {
        double2 *__restrict__ U = a.U + by * a.s_U + off;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int mpv = mpb + r;
            if (m < Lj && mpv < Lj) {
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const int n = 2 * k + 1 - (a.N & 1);  // the carried orders: N + n odd
                    const int i = slot * K + k;
                    const double Er = acc[r][0][i][0], Ei = acc[r][0][i][1];
                    const double Or = acc[r][1][i][0], Oi = acc[r][1][i][1];
                    const int nip = (n + a.N - 1) >> 1;
                    U[((size_t)nip * Lj + m) * Lj + mpv] = rot_i(make_double2(Er + Or, Ei + Oi), n - m + a.eoff);
                    if (n != 0) {
                        const int nim = (-n + a.N - 1) >> 1;
                        double2 dd = make_double2(Er - Or, Ei - Oi);
                        if (mpv & 1) dd = make_double2(-dd.x, -dd.y);
                        U[((size_t)nim * Lj + m) * Lj + mpv] = rot_i(dd, -n - m + a.eoff);
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int k = 0; k < K; ++k) acc[r][q][slot * K + k][0] = acc[r][q][slot * K + k][1] = 0.0;
        }
    };
    // the blocks up to a segment's end, then its flushes; HEAD: until every lane has started.
    // Returns whether the last segment ended.
    auto phase = [&](auto head_c) {
        constexpr bool HEAD = decltype(head_c)::value;
        for (;;) {
            bool last;
            do last = block(head_c);
            while (!last && !(HEAD && lb > lhead));
            if (last) {
                if (sg.Le > 0) flush(0, sg.Le, sg.offe);
                if (sg.Lo > 0) flush(1, sg.Lo, sg.offo);
                if (sgn.s1 == 0) return true;
                if (!HEAD && (sg.s1 & 7)) w.restore(&lds->saved[wave]);
                lo = sg.s1;
                sg = sgn;
                sgn = seg_of(a.segs, ++si + 1);
            }
            if (HEAD && lb > lhead) return false;
        }
    };
    lds_barrier();  // an earlier tile's values are no longer read (persistent executor)
#pragma unroll
    for (int i = 0; i < NS - 1; ++i) request(blk + i, i);
    wait_lds<kLoads * (NS - 2)>();
    lds_barrier();
    load_f(0, 0, 0);
    w.first(0);
    if (!phase(std::true_type())) phase(std::false_type());
    wait_lds<0>();  // the blocks requested beyond the last one: LDS is not written after the tile
}

// ------------------------------------------------------------------------------ synthesis

// A wave's slice of a window: the sums (re, im) of eight steps in 64 lanes, or the state of a block
// that is taken twice.
template <int R, typename VT>
constexpr int adj_slice() {
    return 8 * 64 * 2 * (int)sizeof(VT) >= (int)sizeof(WigState<R>) ? 8 * 64
                                                                     : (int)sizeof(WigState<R>) / (2 * (int)sizeof(VT));
}

// FULL: the form for four waves per SIMD (wig_adj_full_kernel): in FP64 one window instead of two, so that
// the LDS of two workgroups fits a CU, and in both types the window sums taken at once.
template <int K, int R, typename VT, int AW, bool FULL = false>
struct alignas(16) WigAdjLds {
    static constexpr bool ONE = FULL && sizeof(VT) == 8;
    static constexpr int SL = ONE ? 8 * 64 : adj_slice<R, VT>();                       // slice of a wave
    static constexpr int ST = ONE ? (int)sizeof(WigState<R>) / (2 * (int)sizeof(VT)) : 0;  // its state, if apart
    VT win[((ONE ? 1 : 2) * SL + ST) * AW][2];  // the windows of eight steps (then the states)
    WigSlots<K, R, VT, 2> s[AW];
};

// Tile bx of map by; thread tid of AW 64 (AW waves, each with R m' slots).
template <int K, int R, bool XN, typename VT, int AW = kAdjWaves, bool FULL = false>
__device__ __forceinline__ void wig_adj_body(const WigAdjArgs &a, WigAdjLds<K, R, VT, AW, FULL> *lds, int bx, int by,
                                             int tid) {
    using Lds = WigAdjLds<K, R, VT, AW, FULL>;
    constexpr bool ONE = Lds::ONE;
    // VT = double (FP64 path) or float (mixed precision: the m'-sum, its products and its
    // accumulation in FP32; the Delta recursion stays FP64)
    using VC = typename std::conditional<sizeof(VT) == 8, double2, float2>::type;
    typedef VT vc2 __attribute__((ext_vector_type(2)));
    constexpr int SL = Lds::SL;
    // steps pt is loaded ahead (fewer where the registers are short)
    constexpr int PF = (sizeof(VT) == 8 ? K * R >= 8 : K == 6 || (FULL && K > 6)) ? 4 : 8;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
    const int4 t = uniform_tile(a.tiles + bx);
    const int L = a.L, Lp = a.Lp;
    const int m = t.x + lane;
    const int mpb = t.y + wave * R;
    const int wg_start = max(t.x, t.y);                 // smallest l with a non-zero term in the group
    const int lhead = min(L - 1, max(t.x + 63, t.y + AW * R - 1));  // of every wave of the workgroup
    vc2 *const win = (vc2 *)&lds->win[0][0];
    // the saved state of the wave: in its slice of window b, which is free then, or apart
    auto state = [&](int b) { return (WigState<R> *)(win + (ONE ? AW * SL + wave * Lds::ST : (b * AW + wave) * SL)); };

    WigRows<K, R, XN, VT, 2> w;
    w.init(a.seed, a.seedm, a.seede, L, Lp, a.kstride, a.ustride, m, mpb, lane, &lds->s[wave]);
    // The wave's table values: requested two blocks ahead, written to its LDS slots one block
    // ahead (its LDS operations complete in order: no barrier).
    const __amdgpu_buffer_rsrc_t tb = buf_of((const VT *)a.kb2 + (size_t)w.mp0 * a.kstride);
    const __amdgpu_buffer_rsrc_t ub = buf_of(a.uv + (size_t)w.mp0 * a.ustride);
    u32x4 gt, gu;
    auto fetch = [&](int blk) {
        gt = buf_b128(tb, w.to, (unsigned)blk * (16 * K * (unsigned)sizeof(VT)));
        gu = buf_b128(ub, w.uo, (unsigned)blk * 64u);
    };
    auto put = [&](int s) {
        if (lane < w.kTabLanes) ((u32x4 *)&w.sl->tab[s][0][0])[lane] = gt;
        if (lane < w.kULanes) ((u32x4 *)&w.sl->u[s][0][0])[lane] = gu;
    };
    // folded quadrature values of the two active scales: pv[r][l parity][scale slot, k][re, im]
    VT pv[R][2][2 * K][2];
    auto load_slot = [&](int slot, int Lj, long long off) {
        const VC *V = (const VC *)a.V + by * a.s_V + off;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int mpv = mpb + r;
            const bool ok = m < Lj && mpv < Lj;
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    VC v;
                    v.x = v.y = 0;
                    if (ok) v = V[(((size_t)k * 2 + q) * Lj + m) * Lj + mpv];
                    pv[r][q][slot * K + k][0] = v.x;
                    pv[r][q][slot * K + k][1] = v.y;
                }
        }
    };

    const __amdgpu_buffer_rsrc_t pb = buf_of(a.pq);
    const unsigned po = (unsigned)m * 8u, prow = (unsigned)Lp * 8u;
    double p[PF];
    unsigned roff;  // byte offset of the next row of pt to load (rows as in the analysis)
    auto load_p = [&](int slot) {
        p[slot] = buf_f64(pb, po, roff);
        roff += prow;
    };

    char *__restrict__ out = (char *)((VC *)a.Fpart + by * a.s_F + (size_t)(t.y / a.group) * L * Lp);
    int si = t.z, blk = t.w;
    WigSeg sg = seg_of(a.segs, si), sgn = seg_of(a.segs, si + 1);
    int lo = max(sg.s0, wg_start);
    int lb = lo & ~7;
    int buf = 0;
    // PIPE: the sum of a window's slices, in a fixed order (a pairwise tree over the waves: the result
    // does not depend on timing), is taken during the next block, one slice per step, so that
    // its LDS reads run beside the multiply-adds (summed at once after the barrier, all waves
    // read together and nothing else ran).  Not with four slots of two orders in FP64, whose
    // registers are all taken, nor in the FULL form, where the CU's other workgroup runs beside it.
    // A wave sums the rows wave, wave + AW, ..; the window's block starts at plb, its rows
    // pl0 <= l - plb < pl1 are stored.
    constexpr bool PIPE = !FULL && !(sizeof(VT) == 8 && K == 2 && R == 4);
    int plb = 0, pl0 = 0, pl1 = 0;
    vc2 part[3];
    auto sum_store = [&](int li, vc2 v) {
        if (li >= pl0 && li < pl1) {
            // streamed out (read back only by the final reduction): non-temporal, so that the
            // partial sums do not push the tables and V out of L2.  The offset from the
            // workgroup's slice is below 2^32 bytes (one slice is L Lp entries).
            const unsigned off = ((unsigned)(plb + li) * (unsigned)Lp + (unsigned)m) * (unsigned)sizeof(vc2);
            __builtin_nontemporal_store(v, (vc2 *)(out + off));
        }
    };
    auto sum_add = [&](auto s_c, vc2 v) {  // slice S % AW of row wave + AW (S / AW)
        constexpr int S = decltype(s_c)::value, I = S % AW;
        if constexpr ((I & 1) != 0) v = part[0] + v;
        else part[0] = v;
        if constexpr ((I & 3) == 3) v = part[1] + v;
        else if constexpr ((I & 3) == 1) part[1] = v;
        if constexpr (AW == 8) {
            if constexpr (I == 7) v = part[2] + v;
            else if constexpr (I == 3) part[2] = v;
        }
        if constexpr (I == AW - 1) sum_store(wave + AW * (S / AW), v);
    };
    static_assert(AW == 4 || AW == 8, "a wave sums 8 / AW rows of AW slices");
    auto sum_slot = [&](const vc2 *w0, int S) { return w0[(S % AW) * SL + (wave + AW * (S / AW)) * 64 + lane]; };
    auto sum_now = [&] {
        const vc2 *w0 = win + (ONE ? 0 : buf ^ 1) * (AW * SL);
        eight([&](auto s_c) { sum_add(s_c, sum_slot(w0, decltype(s_c)::value)); });
        pl1 = pl0;
    };

    // The block of steps lb .. lb + 7 (table block blk), each wave into its slice of the window;
    // returns whether it ends the segment, and moves on to the next block: the same steps again
    // where the segment ends inside it, from the state at its start.  HEAD as in the analysis.
    auto block = [&](auto head_c) {
        constexpr bool HEAD = decltype(head_c)::value;
        const bool last = lb + 8 >= sg.s1;
        if (!HEAD && last && (sg.s1 & 7)) {
            // the state goes to the wave's slice of the other window, once its sums are read; the
            // next block restores it before it writes there
            if constexpr (PIPE) sum_now();
            if constexpr (!ONE) lds_barrier();
            w.save(state(buf ^ 1));
        }
        vc2 *const slice = win + (buf * AW + wave) * SL + lane;
        const vc2 *const w0 = win + (buf ^ 1) * (AW * SL);
        const int nxt = (blk + 1) & 1;
        put(nxt);
        fetch(blk + 2);
        eight([&](auto s_c) {
            constexpr int S = decltype(s_c)::value;
            vc2 q;
            if constexpr (PIPE) q = sum_slot(w0, S);
            if (!HEAD || (lb + S >= lo && lb + S < sg.s1)) {
                if constexpr (HEAD) w.template start<S>(lb + S);
                VT fr = 0, fi = 0;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    double &F0 = (S & 1) ? w.F1[r] : w.F0[r];
                    const double F1 = (S & 1) ? w.F0[r] : w.F1[r];
                    const VT x = (VT)(XN ? F1 * w.scl[r] : F1);
                    wig_adj_step<K, S>(pv[r][S & 1], F0, F1, x, p[S % PF], w.u[r], w.tab[r], fr, fi);
                }
                vc2 o;
                o.x = fr;
                o.y = fi;
                slice[S * 64] = o;
            }
            load_p(S % PF);
            w.template roll<S, 0>(nxt);
            if constexpr (PIPE) sum_add(s_c, q);
            __builtin_amdgcn_sched_barrier(0);
        });
        if (!HEAD || !last || !(sg.s1 & 7)) w.renorm();
        w.advance();
        // one barrier per window: the window written next was read before it (two with one window)
        lds_barrier();
        plb = lb;
        pl0 = max(lo - lb, 0);
        pl1 = min(sg.s1 - lb, 8);
        if constexpr (!ONE) buf ^= 1;
        if constexpr (!PIPE) sum_now();
        if constexpr (ONE) lds_barrier();  // read before the next block writes it
        ++blk;
        lb = last ? sg.s1 & ~7 : lb + 8;
        return last;
    };
    auto phase = [&](auto head_c) {  // as in the analysis
        constexpr bool HEAD = decltype(head_c)::value;
        for (;;) {
            bool last;
            do last = block(head_c);
            while (!last && !(HEAD && lb > lhead));
            if (last) {
                if (sgn.s1 == 0) return true;
                if (!HEAD && (sg.s1 & 7)) w.restore(state(buf));
                lo = sg.s1;
                sg = sgn;
                sgn = seg_of(a.segs, ++si + 1);
                if (sg.newe) load_slot(0, sg.Lae, sg.offae);
                if (sg.newo) load_slot(1, sg.Lao, sg.offao);
            }
            if (HEAD && lb > lhead) return false;
        }
    };

    lds_barrier();  // the window may hold values of an earlier tile (persistent executor)
    fetch(blk);
    roff = (unsigned)blk * 8u * prow;
#pragma unroll
    for (int s = 0; s < PF; ++s) load_p(s);
    load_slot(0, sg.Lae, sg.offae);
    load_slot(1, sg.Lao, sg.offao);
    put(blk & 1);
    fetch(blk + 1);
    w.first(blk & 1);
    if (!phase(std::true_type())) phase(std::false_type());
    if constexpr (PIPE) sum_now();
}

// One launch per direction: the first nplain workgroups take tiles whose start values
// are normal doubles, the rest take the extended-exponent tiles.
template <int K, int R>
__global__ void __launch_bounds__(256, 2) wig_fwd_kernel(const WigFwdArgs a) {
    __shared__ WigFwdLds<K, R> lds;
    if ((int)blockIdx.x < a.nplain) wig_fwd_body<K, R, false>(a, &lds, blockIdx.x, blockIdx.y, threadIdx.x);
    else wig_fwd_body<K, R, true>(a, &lds, blockIdx.x, blockIdx.y, threadIdx.x);
}

// Waves per SIMD of the synthesis kernel: the LDS of two workgroups of FP32 sums fits a CU, and so
// do their registers (128) up to four values per wave, six in one slot.
template <int K, int R, typename VT>
constexpr int wig_adj_min_waves() { return sizeof(VT) == 4 && (K * R <= 4 || (R == 1 && K <= 6)) ? 4 : 2; }

template <int K, int R, typename VT>
__global__ void __launch_bounds__(kAdjThreads, (wig_adj_min_waves<K, R, VT>())) wig_adj_kernel(const WigAdjArgs a) {
    __shared__ WigAdjLds<K, R, VT, kAdjWaves> lds;
    if ((int)blockIdx.x < a.nplain) wig_adj_body<K, R, false, VT>(a, &lds, blockIdx.x, blockIdx.y, threadIdx.x);
    else wig_adj_body<K, R, true, VT>(a, &lds, blockIdx.x, blockIdx.y, threadIdx.x);
}

// One slot per wave, FULL form: four waves per SIMD where the kernel above has two (in FP64 its two
// windows fill a CU's LDS, in FP32 with seven and eight orders its registers).  Same sums in the same
// order.  For launches with more workgroups than CUs; up to that the kernel above is as fast or faster.
template <int K, typename VT>
__global__ void __launch_bounds__(kAdjThreads, 4) wig_adj_full_kernel(const WigAdjArgs a) {
    __shared__ WigAdjLds<K, 1, VT, kAdjWaves, true> lds;
    if ((int)blockIdx.x < a.nplain)
        wig_adj_body<K, 1, false, VT, kAdjWaves, true>(a, &lds, blockIdx.x, blockIdx.y, threadIdx.x);
    else wig_adj_body<K, 1, true, VT, kAdjWaves, true>(a, &lds, blockIdx.x, blockIdx.y, threadIdx.x);
}

}  // namespace s2dw
