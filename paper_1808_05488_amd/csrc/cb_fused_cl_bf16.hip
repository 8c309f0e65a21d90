// The channel-last fused kernel for bfloat16 (cb_fused_cl.h).
#include "cb_fused_cl.h"

namespace cb {

hipError_t launch_fused_bf16_cl(const Geom& g, const FusedPlan& plan, const uint16_t* shadow, const int32_t* idx,
                                const int* count, const void* KF, const float* bias, int relu, uint16_t* OUT, uint16_t* OUT2,
                                const ClWork& work, hipStream_t st, Tm tm)
{
    return launch_fused_cl<uint16_t>(g, plan, shadow, idx, count, KF, nullptr, bias, relu, OUT, OUT2, work, st, tm);
}

}  // namespace cb
