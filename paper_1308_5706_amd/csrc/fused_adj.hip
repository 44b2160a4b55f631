// Launcher of the fused alpha and gamma kernels (fused_k.h), synthesis.
#include "fused_k.h"

namespace s2dw {

template <class C, int P, int NH, int KS>
static hipError_t launch_ks(const StageArgs &a, const ScaleRefs &refs, int nwg, int maps, hipStream_t st) {
    const dim3 grid((unsigned)nwg, (unsigned)maps), nt((unsigned)(ag_orders<C, P, NH, KS>() * (P / kRM)));
    hipLaunchKernelGGL((gamma_alpha_adj_fft_kernel<C, P, NH, KS>), grid, nt, 0, st, a, refs);
    return hipGetLastError();
}

template <class C, int P, int NH>
static hipError_t launch_nh(const StageArgs &a, const ScaleRefs &refs, int nwg, int maps, hipStream_t st) {
    return 2 * a.L - 1 <= P / 2 ? launch_ks<C, P, NH, 4>(a, refs, nwg, maps, st)
                                : launch_ks<C, P, NH, 8>(a, refs, nwg, maps, st);
}

template <class C, int P>
static hipError_t launch_p(const StageArgs &a, const ScaleRefs &refs, int nwg, int maps, hipStream_t st) {
    switch (a.Nh) {
        case 1: return launch_nh<C, P, 1>(a, refs, nwg, maps, st);
        case 2: return launch_nh<C, P, 2>(a, refs, nwg, maps, st);
        case 3: return launch_nh<C, P, 3>(a, refs, nwg, maps, st);
        case 4: return launch_nh<C, P, 4>(a, refs, nwg, maps, st);
        default: return hipErrorInvalidValue;
    }
}

template <class C>
static hipError_t launch_c(const StageArgs &a, const ScaleRefs &refs, int nwg, int P, int maps, hipStream_t st) {
    switch (P) {
        case 128: return launch_p<C, 128>(a, refs, nwg, maps, st);
        case 256: return launch_p<C, 256>(a, refs, nwg, maps, st);
        case 512: return launch_p<C, 512>(a, refs, nwg, maps, st);
        case 1024: return launch_p<C, 1024>(a, refs, nwg, maps, st);
        case 2048: return launch_p<C, 2048>(a, refs, nwg, maps, st);
        case 4096: return launch_p<C, 4096>(a, refs, nwg, maps, st);
        case 8192: return launch_p<C, 8192>(a, refs, nwg, maps, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_gamma_alpha_adj_fft(const StageArgs &a, const ScaleRefs &refs, int nwg, int P, int maps, hipStream_t st) {
    if (t_rec) return hipErrorNotSupported;
    const int T = 2 * a.L - 1;
    if (refs.n < 1 || refs.n > kMaxScales || nwg < 1 || maps < 1 || a.nb < 1 || a.G < 1 || T > P) return hipErrorInvalidValue;
    for (int i = 0; i < refs.n; ++i)
        if (refs.s[i].Lj < 1 || T + 2 * refs.s[i].Lj - 2 > P || (i > 0 && refs.s[i].first <= refs.s[i - 1].first))
            return hipErrorInvalidValue;
    return a.f32 ? launch_c<float2>(a, refs, nwg, P, maps, st) : launch_c<double2>(a, refs, nwg, P, maps, st);
}

}  // namespace s2dw
