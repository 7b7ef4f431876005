// Instantiations of the F-COO tile kernel: bfloat16 rows shorter than a lane's vector.
#include "fcoo_seg_dispatch.h"

namespace fcoo {
hipError_t seg_launch_bf16_narrow(const SegLaunch &L, bool resid, hipStream_t s)
{
    return resid ? seg_dispatch_narrow<dev::bf16raw, true>(L, s) : seg_dispatch_narrow<dev::bf16raw, false>(L, s);
}
}  // namespace fcoo
