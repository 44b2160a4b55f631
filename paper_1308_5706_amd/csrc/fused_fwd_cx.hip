// The fused alpha and gamma kernels (fused_k.h) of the analysis, complex signals.
#include "fused_k.h"

namespace s2dw {
template hipError_t launch_fused_fft<true, 2>(const StageArgs &, const ScaleRefs &, int, int, int, hipStream_t);
}  // namespace s2dw
