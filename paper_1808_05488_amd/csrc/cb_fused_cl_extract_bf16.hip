#include "cb_fused_cl_extract.h"

namespace cb {

hipError_t launch_fused_bf16_cl_extract(const Geom& g, const FusedPlan& plan, const uint16_t* shadow, const int32_t* idx, const int* count,
                                     const void* KF, const float* bias, int relu, uint16_t* OUT, uint16_t* OUT2,
                                     const ClWork& work, const ExtractJob& job, hipStream_t st, Tm tm)
{
    return launch_fused_cl_extract<uint16_t>(g, plan, shadow, idx, count, KF, nullptr, bias, relu, OUT, OUT2, work, job, st, tm);
}

}  // namespace cb
