// Instantiations of the F-COO tile kernel: float32 rows shorter than a lane's vector.
#include "fcoo_seg_dispatch.h"

namespace fcoo {
hipError_t seg_launch_f32_narrow(const SegLaunch &L, bool resid, hipStream_t s)
{
    return resid ? seg_dispatch_narrow<float, true>(L, s) : seg_dispatch_narrow<float, false>(L, s);
}
}  // namespace fcoo
