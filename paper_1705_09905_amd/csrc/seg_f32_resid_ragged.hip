// Instantiations of the F-COO tile kernel: float factors, fused residual, ranks no multiple of the vector.
#include "fcoo_seg_dispatch.h"

namespace fcoo {
hipError_t seg_launch_f32_resid_ragged(const SegLaunch &L, hipStream_t s) { return seg_dispatch<float, true, true>(L, s); }
}  // namespace fcoo
