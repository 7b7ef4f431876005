// Instantiations of the F-COO tile kernel: dev::bf16raw factors, fused residual, ranks no multiple of the vector.
#include "fcoo_seg_dispatch.h"

namespace fcoo {
hipError_t seg_launch_bf16_resid_ragged(const SegLaunch &L, hipStream_t s) { return seg_dispatch<dev::bf16raw, true, true>(L, s); }
}  // namespace fcoo
