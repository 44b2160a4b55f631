// The alpha and gamma sums of a scale in one kernel where its alpha transforms are chirp
// convolutions: analysis Ub -> W, synthesis W -> G, one beta ring per workgroup, several scales in
// one launch; of a complex signal (M = 2) both real maps, whose sums are the (re, im) pairs of W.
//
// The alpha outputs of a ring never go to memory: as two passes, Y (or X) was written and read
// again, 32 Nh bytes per sample in FP64 next to the 8 G of W (at N = 8 as many), and each scale
// took two launches.  What bounds it up to L of a few hundred is the latency of a convolution
// (eight barriers), so NO orders n >= 0 of the ring run side by side on P/8 threads each, an LDS
// column per order; no more of them (ag_orders), so that several workgroups share a CU and
// one's loads and gamma sums overlap the others' transforms.  A thread owns the samples
// x = tid + k NO P/8 for the gamma sums; where the orders take several passes, those of the
// earlier (analysis) or later ones (synthesis) wait in registers.  Every value is computed by the
// same operations in the same order as by the two-pass kernels.  Measured at L = 256, N = 8 (five
// scales): the two passes took 70 + 50 us in the analysis, this kernel 58 in one launch; the
// synthesis 61 + 65 against 63.
#pragma once

#include <type_traits>

#include "stages_k.h"

namespace s2dw {

// Orders per pass for NH of them: as many as make a workgroup of 256 threads (FP32: 128, its
// shorter transforms leave room for more rings), 512 where a thread would own eight samples of
// every order (their registers).  Measured, ms: round trip L = 256, N = 8, 512 threads 0.357,
// 256 0.344, 128 0.345; multiresolution L = 768, N = 8, 256 1.99, 128 2.02; 32 maps of L = 128,
// N = 8, mixed, 256 1.040, 128 1.002; synthesis L = 421, N = 6 (eight samples), 256 0.386, 512
// 0.369; L = 1500, N = 8 (eight samples, P = 4096: 39 registers spilled with one order a pass,
// hence two) 15.4 against 14.2.
// A complex signal has twice the orders and takes twice the threads from P = 2048 on, for their
// registers.
template <class C, int P, int NH, int KS, int M>
constexpr int ag_orders() {
    if (M == 1 && P >= 4096) return KS == 8 && NH >= 3 && P == 4096 ? 2 : 1;
    if (P >= 4096) return P == 4096 ? 2 : 1;
    const int fit = (KS == 8 ? 512 : (sizeof(C) == 8 ? 128 : 256)) * (M == 2 && P == 2048 ? 2 : 1) / (P / kRM);
    return fit < 1 ? 1 : (fit < M * NH ? fit : M * NH);
}

// KS P/8 samples hold T: KS = 4 (T <= P / 2: the first pass of the transforms skips its zero
// half, also the analysis's, 2Lj - 1 <= T) or 8.
template <class C, int P, int NH, int KS, int M>
__global__ void __launch_bounds__((ag_orders<C, P, NH, KS, M>() * (P / kRM)), kMinWaves)
alpha_gamma_fwd_fft_kernel(const StageArgs a, const ScaleRefs refs) {
    static_assert(kRM == 8 && fft::Plan<P, kRM>::NPASS >= 2, "inputs are read before the column is written");
    using R = real_t<C>;
    constexpr int NV = M * NH;  // orders of the signal's real maps
    constexpr int NO = ag_orders<C, P, NH, KS, M>(), NP = (NV + NO - 1) / NO, NT = P / kRM, NTH = NO * NT;
    constexpr int KT = (KS + NO - 1) / NO, NW = (NP - 1) * NO;  // samples per thread, waiting orders
    __shared__ C cols[NO][fft::padded(P)];
    const int o = threadIdx.x / NT, tid = threadIdx.x - o * NT;
    const ScaleRef &sr = refs.s[ref_of(refs, blockIdx.x)];
    const int Lj = sr.Lj, T = 2 * a.L - 1, N = a.N, nb = a.nb;
    const int b = xcd_column(blockIdx.x - sr.first, nb);
    if (b >= nb) return;
    const C *__restrict__ U0 = (const C *)a.in + blockIdx.y * M * a.s_in + sr.in_off + b;
    const C *__restrict__ csq = (const C *)a.csq;
    const int Na = 2 * Lj - 1;
    C held[NW > 0 ? NW : 1][KT];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int v = min(p * NO + o, NV - 1);  // past the last order: its column is not read
        const int np = M == 1 ? v : v % NH;
        const C *__restrict__ U = M == 1 ? U0 : U0 + (v / NH) * a.s_in;
        const int ni = (N / 2) + np, nj = N - 1 - ni;  // rows of n >= 0 and of -n
        const bool zero_n = ni == nj;
        const C *__restrict__ Up = U + (size_t)ni * Lj * nb;
        const C *__restrict__ Um = U + (size_t)nj * Lj * nb;
        auto in = [&](int i, int = 0) {  // branch-free (see alpha_fwd_fft_body)
            const bool ok = i < Na;
            const int m = (ok ? i : Na - 1) - (Lj - 1), am = m < 0 ? -m : m;
            C c = (m >= 0 ? Up : Um)[(size_t)am * nb];
            const C w = csq[am];
            if (m < 0) c = cconj(c);
            if (m == 0 && zero_n) c.y = 0.0;
            c = cmul(c, w);
            return ok ? c : zero2<C>();
        };
        C *col = cols[o];
        auto st = [&](int i, C v, int = 0) {
            const int x = i - (Na - 1);
            if (x >= 0 && x < T) col[pad(x)] = cmul(v, csq[x]);
        };
        fft::convolve_io<P, kRM, (KS == 4 ? 1 : -1)>(col, tid, (const C *)a.tw, (const C *)sr.hh, in, st, Na);
        if (p < NP - 1) {
            // read before the next transform's first barrier, and it writes the columns after that
#pragma unroll
            for (int q = 0; q < NO; ++q)
#pragma unroll
                for (int k = 0; k < KT; ++k) {
                    const int x = threadIdx.x + k * NTH;
                    if (x < T) held[p * NO + q][k] = cols[q][pad(x)];
                }
        }
    }
    using WT = std::conditional_t<M == 2, C, R>;
    WT *__restrict__ W = (WT *)a.wout + blockIdx.y * a.s_w + sr.out_off + (size_t)b * T;
    const UniTab<C> tg(a.tg);
    const size_t plane = (size_t)nb * T;
    const int G = a.G;
#pragma unroll
    for (int k = 0; k < KT; ++k) {
        const int x = threadIdx.x + k * NTH;
        if (x >= T) continue;
        C y[NV];
#pragma unroll
        for (int r = 0; r < NV; ++r) y[r] = r < NW ? held[r < NW ? r : 0][k] : cols[r < NW ? 0 : r - NW][pad(x)];
        for_gamma<NH>(tg, G, [&](int g, const C *w) {
            R acc[M];
#pragma unroll
            for (int c = 0; c < M; ++c) acc[c] = 0;
#pragma unroll
            for (int r = 0; r < NH; ++r)
#pragma unroll
                for (int c = 0; c < M; ++c)
                    acc[c] = fma(y[c * NH + r].x, w[r].x, fma(-y[c * NH + r].y, w[r].y, acc[c]));
            if constexpr (M == 2) nt_store(mk<C>(acc[0], acc[M - 1]), W + g * plane + x);
            else __builtin_nontemporal_store(acc[0], W + g * plane + x);
        });
    }
}

template <class C, int P, int NH, int KS, int M>
__global__ void __launch_bounds__((ag_orders<C, P, NH, KS, M>() * (P / kRM)), kMinWaves)
gamma_alpha_adj_fft_kernel(const StageArgs a, const ScaleRefs refs) {
    static_assert(kRM == 8 && fft::Plan<P, kRM>::NPASS >= 2, "inputs are read before the column is written");
    using R = real_t<C>;
    constexpr int NV = M * NH;  // orders of the signal's real maps
    constexpr int NO = ag_orders<C, P, NH, KS, M>(), NP = (NV + NO - 1) / NO, NT = P / kRM, NTH = NO * NT;
    constexpr int KT = (KS + NO - 1) / NO;
    __shared__ C cols[NO][fft::padded(P)];
    const int o = threadIdx.x / NT, tid = threadIdx.x - o * NT;
    const ScaleRef &sr = refs.s[ref_of(refs, blockIdx.x)];
    const int Lj = sr.Lj, T = 2 * a.L - 1, N = a.N, nb = a.nb, G = a.G;
    const int b = xcd_column(blockIdx.x - sr.first, nb);
    if (b >= nb) return;
    using WT = std::conditional_t<M == 2, C, R>;
    const WT *__restrict__ W = (const WT *)a.win + blockIdx.y * a.s_w + sr.in_off + (size_t)b * T;
    const UniTab<C> tg(a.tg);
    const C *__restrict__ csq = (const C *)a.csq;
    const size_t plane = (size_t)nb * T;
    // the gamma sums of every order at the owned samples (those past the end repeat the last:
    // their sums are not used)
    C x[NV][KT];
#pragma unroll
    for (int r = 0; r < NV; ++r)
#pragma unroll
        for (int k = 0; k < KT; ++k) x[r][k] = zero2<C>();
    // eight samples requested at a time
#pragma unroll (KT >= 8 ? 1 : 8 / KT)
    for (int g = 0; g < G; ++g) {
        R w[M][KT];
#pragma unroll
        for (int k = 0; k < KT; ++k) {
            const WT *p = W + g * plane + min((int)threadIdx.x + k * NTH, T - 1);
            if constexpr (M == 2) {
                const C z = nt_load(p);
                w[0][k] = z.x;
                w[M - 1][k] = z.y;
            } else {
                w[0][k] = __builtin_nontemporal_load(p);
            }
        }
#pragma unroll
        for (int r = 0; r < NH; ++r) {
            const C t = tg[g * NH + r];
#pragma unroll
            for (int c = 0; c < M; ++c)
#pragma unroll
                for (int k = 0; k < KT; ++k) {
                    C &z = x[c * NH + r][k];
                    z.x = fma(w[c][k], t.x, z.x);
                    z.y = fma(w[c][k], t.y, z.y);
                }
        }
    }
    const int Nk = 2 * Lj - 1;
    const R s = (R)a.scale;
    C *__restrict__ Go = (C *)a.out + blockIdx.y * M * a.s_out + sr.out_off + b;
    C *col = cols[o];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const bool live = p * NO + o < NV;
        const int v = live ? p * NO + o : NV - 1;
        const int np = M == 1 ? v : v % NH;
        C *__restrict__ Gv = M == 1 ? Go : Go + (v / NH) * a.s_out;
        const int ni = (N / 2) + np, nj = N - 1 - ni;
        const bool zero_n = ni == nj;
        C *__restrict__ Gp = Gv + (size_t)ni * Lj * nb;
        C *__restrict__ Gm = Gv + (size_t)nj * Lj * nb;
        if constexpr (NO > 1) {
            // the columns are free: each transform ends with a barrier
#pragma unroll
            for (int q = 0; q < NO; ++q)
#pragma unroll
                for (int k = 0; k < KT; ++k) {
                    const int i = threadIdx.x + k * NTH;
                    if (i < T) cols[q][pad(i)] = x[p * NO + q < NV ? p * NO + q : NV - 1][k];
                }
            __syncthreads();
        }
        auto in = [&](int i, int slot) {  // slot k of the first pass is the sample tid + k NT
            const bool ok = i < T;
            const int ic = ok ? i : T - 1;
            C u;
            if constexpr (NO > 1) u = col[pad(ic)];
            else u = x[p][slot < KT ? slot : KT - 1];
            const C v = cmulc(u, csq[ic]);
            return ok ? v : zero2<C>();
        };
        auto st = [&](int i, C v, int = 0) {
            const int q = i - (T - 1);
            if (q >= 0 && q < Nk && live) {
                const int m = q - (Lj - 1);
                const C z = cscale(cmulc(v, csq[m < 0 ? -m : m]), s);
                if (m >= 0) Gp[(size_t)m * nb] = z;
                if (m <= 0 && !zero_n) Gm[(size_t)(-m) * nb] = cconj(z);
            }
        };
        fft::convolve_io<P, kRM, (KS == 4 ? 1 : 0)>(col, tid, (const C *)a.tw, (const C *)sr.hh, in, st, T);
    }
}

// ------------------------------------------------------------------------------ launcher

template <bool FWD, class C, int P, int NH, int KS, int M>
static hipError_t fused_launch(const StageArgs &a, const ScaleRefs &refs, int nwg, int signals, hipStream_t st) {
    // (the forms that fused_fft refuses)
    if constexpr (M == 2 && P >= 4096 && NH > 2 && (P == 8192 || KS == 8)) {
        return hipErrorInvalidValue;
    } else {
        const dim3 grid((unsigned)nwg, (unsigned)signals), nt((unsigned)(ag_orders<C, P, NH, KS, M>() * (P / kRM)));
        if constexpr (FWD) hipLaunchKernelGGL((alpha_gamma_fwd_fft_kernel<C, P, NH, KS, M>), grid, nt, 0, st, a, refs);
        else hipLaunchKernelGGL((gamma_alpha_adj_fft_kernel<C, P, NH, KS, M>), grid, nt, 0, st, a, refs);
        return hipGetLastError();
    }
}

template <bool FWD, class C, int P, int M>
static hipError_t fused_orders(const StageArgs &a, const ScaleRefs &refs, int nwg, int signals, hipStream_t st) {
    const bool low = 2 * a.L - 1 <= P / 2;
    switch (a.Nh) {
#define S2DW_FUSED_NH(NH)                                                                 \
    case NH:                                                                              \
        return low ? fused_launch<FWD, C, P, NH, 4, M>(a, refs, nwg, signals, st)         \
                   : fused_launch<FWD, C, P, NH, 8, M>(a, refs, nwg, signals, st);
        S2DW_FUSED_NH(1)
        S2DW_FUSED_NH(2)
        S2DW_FUSED_NH(3)
        S2DW_FUSED_NH(4)
#undef S2DW_FUSED_NH
        default: return hipErrorInvalidValue;
    }
}

template <bool FWD, class C, int M>
static hipError_t fused_size(const StageArgs &a, const ScaleRefs &refs, int nwg, int P, int signals, hipStream_t st) {
    switch (P) {
        case 128: return fused_orders<FWD, C, 128, M>(a, refs, nwg, signals, st);
        case 256: return fused_orders<FWD, C, 256, M>(a, refs, nwg, signals, st);
        case 512: return fused_orders<FWD, C, 512, M>(a, refs, nwg, signals, st);
        case 1024: return fused_orders<FWD, C, 1024, M>(a, refs, nwg, signals, st);
        case 2048: return fused_orders<FWD, C, 2048, M>(a, refs, nwg, signals, st);
        case 4096: return fused_orders<FWD, C, 4096, M>(a, refs, nwg, signals, st);
        case 8192: return fused_orders<FWD, C, 8192, M>(a, refs, nwg, signals, st);
        default: return hipErrorInvalidValue;
    }
}

template <bool FWD, int M>
hipError_t launch_fused_fft(const StageArgs &a, const ScaleRefs &refs, int nwg, int P, int signals, hipStream_t st) {
    if (t_rec) return hipErrorNotSupported;
    const int T = 2 * a.L - 1;
    if (refs.n < 1 || refs.n > kMaxScales || nwg < 1 || signals < 1 || a.nb < 1 || a.G < 1 || T > P)
        return hipErrorInvalidValue;
    for (int i = 0; i < refs.n; ++i)
        if (refs.s[i].Lj < 1 || refs.s[i].Lj > a.L || T + 2 * refs.s[i].Lj - 2 > P ||
            (i > 0 && refs.s[i].first <= refs.s[i - 1].first))
            return hipErrorInvalidValue;
    return a.f32 ? fused_size<FWD, float2, M>(a, refs, nwg, P, signals, st)
                 : fused_size<FWD, double2, M>(a, refs, nwg, P, signals, st);
}

}  // namespace s2dw
