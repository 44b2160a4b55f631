// The alpha and gamma sums in one kernel for scales whose alpha transforms are blocked (real
// signals, see alpha_fwd_blk_body): one beta ring per workgroup, several scales in one launch.
//
// As two passes the alpha outputs of these scales, Nh T complex values a ring for a handful of
// coefficients, made a round trip through memory: at L = 1024, N = 8 the blocked alpha pass took
// 64-90 us a scale and the gamma pass 76, W alone 57 at the rate of a fill.  Here the NH orders run
// side by side on P/8 threads each, and the gamma sums of a block of samples are taken as soon as
// it is transformed (analysis), or formed in the columns before it is (synthesis), so nothing
// waits in registers and nothing is staged.  Same operations in the same order as the two passes.
#include "stages_k.h"

namespace s2dw {

template <class C, int P, int NH>
__global__ void __launch_bounds__((NH * (P / kRM)), kMinWaves)
alpha_gamma_fwd_blk_kernel(const StageArgs a, const ScaleRefs refs) {
    static_assert(kRM == 8 && fft::Plan<P, kRM>::NPASS >= 2, "the first pass reads element tid + r NT into slot r");
    using R = real_t<C>;
    constexpr int NT = P / kRM, NTH = NH * NT;
    __shared__ C cols[NH][fft::padded(P)];
    const int np = threadIdx.x / NT, tid = threadIdx.x - np * NT;
    const ScaleRef &sr = refs.s[ref_of(refs, blockIdx.x)];
    const int Lj = sr.Lj, T = 2 * a.L - 1, N = a.N, nb = a.nb, B = sr.B, nblk = sr.nblk, G = a.G;
    const int b = xcd_column(blockIdx.x - sr.first, nb);
    if (b >= nb) return;
    const int ni = (N / 2) + np, nj = N - 1 - ni;
    const bool zero_n = ni == nj;
    const C *__restrict__ Up = (const C *)a.in + blockIdx.y * a.s_in + sr.in_off + (size_t)ni * Lj * nb + b;
    const C *__restrict__ Um = (const C *)a.in + blockIdx.y * a.s_in + sr.in_off + (size_t)nj * Lj * nb + b;
    const C *__restrict__ csq = (const C *)a.csq;
    const C *__restrict__ eph = (const C *)a.eph;
    const int Na = 2 * Lj - 1;
    C base[kRM];
#pragma unroll
    for (int s = 0; s < kRM; ++s) {  // branch-free (see alpha_fwd_fft_body)
        const int i = tid + s * NT;
        const bool ok = i < Na;
        const int m = (ok ? i : Na - 1) - (Lj - 1), am = m < 0 ? -m : m;
        C c = (m >= 0 ? Up : Um)[(size_t)am * nb];
        const C w = csq[am];
        if (m < 0) c = cconj(c);
        if (m == 0 && zero_n) c.y = 0.0;
        c = cmul(c, w);
        base[s] = ok ? c : zero2<C>();
    }
    R *__restrict__ W = (R *)a.wout + blockIdx.y * a.s_w + sr.out_off + (size_t)b * T;
    const UniTab<C> tg(a.tg);
    const size_t plane = (size_t)nb * T;
    C *col = cols[np];
    for (int k = 0; k < nblk; ++k) {
        const int a0 = k * B, nx = min(B, T - a0);
        auto in = [&](int i, int s) {
            int r = ((i - (Lj - 1)) * a0) % T;
            if (r < 0) r += T;
            return cmul(base[s], eph[r]);
        };
        auto st = [&](int i, C v, int = 0) {
            const int x = i - (Na - 1);
            if (x >= 0 && x < nx) col[pad(x)] = cmul(v, csq[x]);
        };
        fft::convolve_io<P, kRM>(col, tid, (const C *)a.tw, (const C *)sr.hh, in, st, Na);
        // the next block writes the columns after its first barrier
        for (int x = threadIdx.x; x < nx; x += NTH) {
            C y[NH];
#pragma unroll
            for (int r = 0; r < NH; ++r) y[r] = cols[r][pad(x)];
            for_gamma<NH>(tg, G, [&](int g, const C *w) {
                R acc = 0;
#pragma unroll
                for (int r = 0; r < NH; ++r) acc = fma(y[r].x, w[r].x, fma(-y[r].y, w[r].y, acc));
                __builtin_nontemporal_store(acc, W + g * plane + a0 + x);
            });
        }
    }
}

template <class C, int P, int NH>
__global__ void __launch_bounds__((NH * (P / kRM)), kMinWaves)
gamma_alpha_adj_blk_kernel(const StageArgs a, const ScaleRefs refs) {
    static_assert(kRM == 8 && fft::Plan<P, kRM>::NPASS >= 2, "the first pass reads every input, then writes");
    using R = real_t<C>;
    constexpr int NT = P / kRM, NTH = NH * NT, KT = (kRM + NH - 1) / NH;  // samples of a block per thread
    __shared__ C cols[NH][fft::padded(P)];
    const int np = threadIdx.x / NT, tid = threadIdx.x - np * NT;
    const ScaleRef &sr = refs.s[ref_of(refs, blockIdx.x)];
    const int Lj = sr.Lj, T = 2 * a.L - 1, N = a.N, nb = a.nb, B = sr.B, nblk = sr.nblk, G = a.G;
    const int b = xcd_column(blockIdx.x - sr.first, nb);
    if (b >= nb) return;
    const int ni = (N / 2) + np, nj = N - 1 - ni;
    const bool zero_n = ni == nj;
    const R *__restrict__ W = (const R *)a.win + blockIdx.y * a.s_w + sr.in_off + (size_t)b * T;
    const UniTab<C> tg(a.tg);
    const C *__restrict__ csq = (const C *)a.csq;
    const C *__restrict__ eph = (const C *)a.eph;
    const size_t plane = (size_t)nb * T;
    const int Nk = 2 * Lj - 1;
    C *col = cols[np];
    C acc[kRM];
    int qs[kRM];
#pragma unroll
    for (int s = 0; s < kRM; ++s) {
        acc[s] = zero2<C>();
        qs[s] = -1;
    }
    for (int k = 0; k < nblk; ++k) {
        const int a0 = k * B, nx = min(B, T - a0);
        {
            C x[NH][KT];
#pragma unroll
            for (int r = 0; r < NH; ++r)
#pragma unroll
                for (int t = 0; t < KT; ++t) x[r][t] = zero2<C>();
#pragma unroll (8 / KT)
            for (int g = 0; g < G; ++g) {
                R w[KT];
#pragma unroll
                for (int t = 0; t < KT; ++t)
                    w[t] = __builtin_nontemporal_load(W + g * plane + a0 + min((int)threadIdx.x + t * NTH, nx - 1));
#pragma unroll
                for (int r = 0; r < NH; ++r) {
                    const C e = tg[g * NH + r];
#pragma unroll
                    for (int t = 0; t < KT; ++t) {
                        x[r][t].x = fma(w[t], e.x, x[r][t].x);
                        x[r][t].y = fma(w[t], e.y, x[r][t].y);
                    }
                }
            }
            // the columns are free: each transform ends with a barrier
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                const int i = threadIdx.x + t * NTH;
                if (i < nx)
#pragma unroll
                    for (int r = 0; r < NH; ++r) cols[r][pad(i)] = x[r][t];
            }
        }
        __syncthreads();
        auto in = [&](int i, int = 0) {
            const bool ok = i < nx;
            const int ic = ok ? i : 0;
            const C v = cmulc(col[pad(ic)], csq[ic]);
            return ok ? v : zero2<C>();
        };
        // the block's part of Zh(m), q = m + Lj - 1 < 2Lj - 1, comes out at q + B - 1
        auto st = [&](int i, C v, int s) {
            const int q = i - (B - 1);
            qs[s] = q;
            if (q >= 0 && q < Nk) {
                const int m = q - (Lj - 1);
                int r = (-m * a0) % T;
                if (r < 0) r += T;
                acc[s] = cadd(acc[s], cmul(cmulc(v, csq[m < 0 ? -m : m]), eph[r]));
            }
        };
        fft::convolve_io<P, kRM>(col, tid, (const C *)a.tw, (const C *)sr.hh, in, st, B);
    }
    const R sc = (R)a.scale;
    C *__restrict__ Gp = (C *)a.out + blockIdx.y * a.s_out + sr.out_off + (size_t)ni * Lj * nb + b;
    C *__restrict__ Gm = (C *)a.out + blockIdx.y * a.s_out + sr.out_off + (size_t)nj * Lj * nb + b;
#pragma unroll
    for (int s = 0; s < kRM; ++s) {
        const int q = qs[s];
        if (q >= 0 && q < Nk) {
            const int m = q - (Lj - 1);
            const C z = cscale(acc[s], sc);
            if (m >= 0) Gp[(size_t)m * nb] = z;
            if (m <= 0 && !zero_n) Gm[(size_t)(-m) * nb] = cconj(z);
        }
    }
}

// ------------------------------------------------------------------------------ launcher

template <bool FWD, class C, int P>
static hipError_t blk_orders(const StageArgs &a, const ScaleRefs &refs, int nwg, int maps, hipStream_t st) {
    const dim3 grid((unsigned)nwg, (unsigned)maps), nt((unsigned)(a.Nh * (P / kRM)));
    switch (a.Nh) {
#define S2DW_BLK_NH(NH)                                                                                            \
    case NH:                                                                                                       \
        if constexpr (FWD) hipLaunchKernelGGL((alpha_gamma_fwd_blk_kernel<C, P, NH>), grid, nt, 0, st, a, refs);   \
        else hipLaunchKernelGGL((gamma_alpha_adj_blk_kernel<C, P, NH>), grid, nt, 0, st, a, refs);                 \
        break;
        S2DW_BLK_NH(1)
        S2DW_BLK_NH(2)
        S2DW_BLK_NH(3)
        S2DW_BLK_NH(4)
#undef S2DW_BLK_NH
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <bool FWD, class C>
static hipError_t blk_size(const StageArgs &a, const ScaleRefs &refs, int nwg, int P, int maps, hipStream_t st) {
    switch (P) {
        case 512: return blk_orders<FWD, C, 512>(a, refs, nwg, maps, st);
        case 1024: return blk_orders<FWD, C, 1024>(a, refs, nwg, maps, st);
        case 2048: return blk_orders<FWD, C, 2048>(a, refs, nwg, maps, st);
        default: return hipErrorInvalidValue;
    }
}

template <bool FWD>
hipError_t launch_fused_blk(const StageArgs &a, const ScaleRefs &refs, int nwg, int P, int maps, hipStream_t st) {
    if (t_rec) return hipErrorNotSupported;
    const int T = 2 * a.L - 1;
    if (refs.n < 1 || refs.n > kMaxScales || nwg < 1 || maps < 1 || a.nb < 1 || a.G < 1) return hipErrorInvalidValue;
    for (int i = 0; i < refs.n; ++i) {
        const ScaleRef &r = refs.s[i];
        if (r.Lj < 1 || r.Lj > a.L || r.B < 1 || r.B + 2 * r.Lj - 2 > P || (long)r.B * r.nblk < T ||
            (long)r.B * (r.nblk - 1) >= T || (i > 0 && r.first <= refs.s[i - 1].first))
            return hipErrorInvalidValue;
    }
    return a.f32 ? blk_size<FWD, float2>(a, refs, nwg, P, maps, st) : blk_size<FWD, double2>(a, refs, nwg, P, maps, st);
}

template hipError_t launch_fused_blk<true>(const StageArgs &, const ScaleRefs &, int, int, int, hipStream_t);
template hipError_t launch_fused_blk<false>(const StageArgs &, const ScaleRefs &, int, int, int, hipStream_t);

}  // namespace s2dw
