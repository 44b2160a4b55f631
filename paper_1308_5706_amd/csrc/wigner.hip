// Launchers of the Wigner-stage kernels (wigner_k.h) and the tile-shape options.
#include "wigner_k.h"

namespace s2dw {

// ------------------------------------------------------------------------------ launchers

template <int K, int R>
static hipError_t launch_fwd_k(const WigFwdArgs &a, int ntiles, int maps, hipStream_t st) {
    if (ntiles <= 0) return hipSuccess;
    hipLaunchKernelGGL((wig_fwd_kernel<K, R>), dim3(ntiles, maps), dim3(256), 0, st, a);
    return hipGetLastError();
}

// More workgroups than CUs: the FULL form of the one-slot synthesis where it has one (FP64: up to two
// orders, whose registers allow it; FP32: from seven on, where the ordinary form has not four waves per
// SIMD already).  Measured, synthesis stage with the final sum, us, ordinary against FULL: 16 maps of L = 128,
// N = 1 65 against 54, 64 maps 216 against 167; 8 maps of L = 256, N = 4 155 against 136; mixed, 8 maps of
// L = 200, N = 16 167 against 131; one map of it 83 against 84, 16 maps of L = 100, N = 4 (416 workgroups)
// 49 against 50.
template <int K, int R, typename VT>
constexpr bool has_full() { return R == 1 && (sizeof(VT) == 8 ? K <= 2 : K >= 7); }

template <int K, int R, typename VT>
static hipError_t launch_adj_t(const WigAdjArgs &a, int ntiles, int maps, hipStream_t st) {
    const dim3 grid(ntiles, maps), nt(kAdjThreads);
    if constexpr (has_full<K, R, VT>()) {
        if ((long)ntiles * maps > 256) {
            hipLaunchKernelGGL((wig_adj_full_kernel<K, VT>), grid, nt, 0, st, a);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((wig_adj_kernel<K, R, VT>), grid, nt, 0, st, a);
    return hipGetLastError();
}

template <int K, int R>
static hipError_t launch_adj_k(const WigAdjArgs &a, int ntiles, int maps, hipStream_t st) {
    if (ntiles <= 0) return hipSuccess;
    return a.f32 ? launch_adj_t<K, R, float>(a, ntiles, maps, st) : launch_adj_t<K, R, double>(a, ntiles, maps, st);
}

// m' slots per wave.  The accumulators (analysis) or quadrature values (synthesis) take 16 R K
// registers, kept at or below 128 for two waves per SIMD.  More slots share the per-lane loads
// and, in the synthesis, the window sums and the partial sums of a group; but below a few waves
// per SIMD (1024 of them) a wave's own chain of steps is what takes the time, and fewer slots
// make it shorter.  Measured (us, one map, FP64; analysis / synthesis with the final sum), slots
// 1, 2, 4: L = 256, N = 8 (1024 waves at one slot) 48, 66 / 91, 114; L = 421, N = 6 (2947) 59, 79 /
// 126, 151; L = 512, N = 4 (4096) 59, 77, 113 / 140, 153, 214; L = 512, N = 1 50, 62, 85 / 128, 126,
// 169; L = 1024, N = 8 (16384) 456, 395 / 830, 596; L = 1024, N = 3 330, 241, 226 / 561, 466, 414;
// L = 2048, N = 4 2206, 1713, 1585 / 4199, 3327, 2569.
static int wig_slots(int K, long waves, long one) {
    const int most = K >= 5 ? 1 : (K >= 3 ? 2 : 4);
    if (waves <= one) return 1;
    return waves <= 12000 && most > 2 ? 2 : most;
}
// One map takes one slot longer than a batch of the same waves, whose chains are shorter (N = 4:
// L = 576, 5184 waves, 72 us with one slot, 86 with two; L = 640 99 and 96; 16 maps of L = 128, 4096
// waves, 51 and 45; 4 of L = 256 56 and 63, 6 of them 73 and 70).
// One order: a batch of small maps takes four slots earlier (24 maps of L = 128: 44 us against 50
// with two; one map of L = 640 71 with two, 99 with four).
int wig_fwd_slots_for(int K, long waves, int maps) {
    return K <= 1 && waves <= 3500 && waves * maps > 6000 ? 4 : wig_slots(K, waves * maps, maps == 1 ? 6000 : 3500);
}
// Mixed precision: one number of slots at every size, so that its FP32 sums over the m' of a group
// are rounded the same way in every call.
// FP64: the number follows the size of a map, not of the batch, whose maps have the results of single
// calls.  One slot is up to 5 % faster for one map and up to 5 % slower for a batch about the line (whole
// syntheses, ms, one and two slots; N = 1: one map of L = 256 0.090, 0.095, 20 maps 0.473, 0.448; one of
// L = 512 0.177, 0.175, 8 maps 0.929, 0.820.  N = 4: one of L = 400 0.275, 0.291, 16 maps 2.62, 2.59;
// one of L = 512 0.347, 0.357, 24 maps 6.43, 6.17; one of L = 600 0.600, 0.612, 8 maps 4.02, 3.93).
int wig_adj_slots(int K, long waves, int f32) {
    if (f32) return K >= 5 ? 1 : (K >= 2 ? 2 : 4);
    return wig_slots(K, waves, K <= 1 ? 1024 : 5000);
}

// Slot counts compiled for each number of carried orders K (the tile shapes the tuner may pick).
int wig_slot_options(int K, int *R) {
    if (K <= 1) {
        R[0] = 1, R[1] = 2, R[2] = 4;
        return 3;
    }
    if (K == 2) {
        R[0] = 1, R[1] = 2, R[2] = 4;
        return 3;
    }
    if (K <= 4) {
        R[0] = 1, R[1] = 2;
        return 2;
    }
    R[0] = 1;
    return 1;
}

#define S2DW_WIG_SWITCH(FN)                                          \
    switch (K * 8 + R) {                                             \
        case 1 * 8 + 1: return FN<1, 1>(a, ntiles, maps, st);        \
        case 1 * 8 + 2: return FN<1, 2>(a, ntiles, maps, st);        \
        case 1 * 8 + 4: return FN<1, 4>(a, ntiles, maps, st);        \
        case 2 * 8 + 1: return FN<2, 1>(a, ntiles, maps, st);        \
        case 2 * 8 + 2: return FN<2, 2>(a, ntiles, maps, st);        \
        case 2 * 8 + 4: return FN<2, 4>(a, ntiles, maps, st);        \
        case 3 * 8 + 1: return FN<3, 1>(a, ntiles, maps, st);        \
        case 3 * 8 + 2: return FN<3, 2>(a, ntiles, maps, st);        \
        case 4 * 8 + 1: return FN<4, 1>(a, ntiles, maps, st);        \
        case 4 * 8 + 2: return FN<4, 2>(a, ntiles, maps, st);        \
        case 5 * 8 + 1: return FN<5, 1>(a, ntiles, maps, st);        \
        case 6 * 8 + 1: return FN<6, 1>(a, ntiles, maps, st);        \
        case 7 * 8 + 1: return FN<7, 1>(a, ntiles, maps, st);        \
        case 8 * 8 + 1: return FN<8, 1>(a, ntiles, maps, st);        \
        default: return hipErrorInvalidValue;                        \
    }

hipError_t launch_wig_fwd(const WigFwdArgs &a, int K, int R, int ntiles, int maps, hipStream_t st) {
    if (t_rec) return K <= 4 ? rec_job(pkind(PS_WIGF, 0, K, R), ntiles, maps, 256, a) : hipErrorNotSupported;
    S2DW_WIG_SWITCH(launch_fwd_k)
}

hipError_t launch_wig_adj(const WigAdjArgs &a, int K, int R, int ntiles, int maps, hipStream_t st) {
    if (t_rec) return K <= 4 ? rec_job(pkind(PS_WIGA, a.f32, K, R), ntiles, maps, 256, a) : hipErrorNotSupported;
    S2DW_WIG_SWITCH(launch_adj_k)
}

}  // namespace s2dw
