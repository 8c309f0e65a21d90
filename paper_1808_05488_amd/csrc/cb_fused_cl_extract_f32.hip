#include "cb_fused_cl_extract.h"

namespace cb {

hipError_t launch_fused_f32_cl_extract(const Geom& g, const FusedPlan& plan, const float* shadow, const int32_t* idx, const int* count,
                                     const void* KF, const float* KT, const float* bias, int relu, float* OUT, float* OUT2,
                                     const ClWork& work, const ExtractJob& job, hipStream_t st, Tm tm)
{
    return launch_fused_cl_extract<float>(g, plan, shadow, idx, count, KF, KT, bias, relu, OUT, OUT2, work, job, st, tm);
}

}  // namespace cb
