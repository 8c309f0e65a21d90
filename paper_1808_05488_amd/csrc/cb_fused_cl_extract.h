// The channel-last fused kernel with the index extraction of the next layer in front (one element type per source file).
#pragma once
#include "cb_extract.h"
#include "cb_fused_cl.h"

namespace cb {

namespace {

// The product with the index extraction of the layer behind it in front: workgroups 0 .. job.nblk - 1 extract (the grid has them rounded
// up to 8, so that the others keep their XCDs), the others multiply.  The extraction alone is a launch of 4 - 7 us in which a handful of
// compute units work, and it needs nothing of the product: frames of the ten-layer trunk of 3 x 3
// filters at 368x656 with propagated change maps, 5 % changed, us: bfloat16 203 -> 157, float32 343 -> 291; of the five-layer 7 x 7 net at
// 480x640 110 -> 97.
template <typename T, int SHAPE, int FAR>
__global__ __launch_bounds__(256, sizeof(T) == 2 ? 4 : 3) void fused_cl_extract_kernel(Geom g, ClDiv div, const T* __restrict__ S2,
                                                          const int32_t* __restrict__ idx, const int* __restrict__ count,
                                                          const uint4* __restrict__ KF, const float* __restrict__ KT,
                                                          const float* __restrict__ bias, int relu,
                                                          T* __restrict__ OUT, T* __restrict__ OUT2, ExtractJob job, float* ws, unsigned ws_bytes, int* kcount)
{
    extern __shared__ uint4 dyn_lds4[];
    static_assert(EXTRACT_LDS <= (sizeof(T) == 4 ? CL_LDS_F32 : CL_LDS_BF16), "the extraction's part of a map fits");
    const unsigned first = ((unsigned)job.nblk + 7u) & ~7u;
    if (blockIdx.x < first) {
        if (blockIdx.x < (unsigned)job.nblk) extract_block(job, (int)blockIdx.x, reinterpret_cast<uint64_t*>(dyn_lds4));
        return;
    }
    fused_cl_run<T, SHAPE, true, FAR>(g, div, S2, idx, count, KF, KT, bias, relu, OUT, OUT2, blockIdx.x - first, CL_GRID, ws, ws_bytes, kcount);
}

template <typename T>
hipError_t launch_fused_cl_extract(const Geom& g, const FusedPlan& plan, const T* shadow, const int32_t* idx, const int* count, const void* KF,
                                   const float* KT, const float* bias, int relu, T* OUT, T* OUT2, const ClWork& work, const ExtractJob& job, hipStream_t st, Tm tm)
{
    if (!fused_takes_job(g, plan) || !extract_fits(job.g) || job.nblk != dilate_num_blocks(job.g)) return hipErrorInvalidValue;
    const ClDiv div = cl_div(g.Wo, g.Ho, g.kw, g.Cs);
    return fused_cl_instance<T>(g, plan, [&](auto shape) {
        constexpr int SHAPE = decltype(shape)::value;
#define CB_CLX(far) \
    CB_LAUNCH_LDS((fused_cl_extract_kernel<T, SHAPE, far>), dim3(CL_GRID + (((unsigned)job.nblk + 7u) & ~7u)), dim3(256), \
                  cl_lds_bytes<T>(), st, tm, g, div, shadow, idx, count, (const uint4*)KF, KT, bias, relu, OUT, OUT2, job, work.ws, work.bytes, work.count)
        const int far = fused_cl_far_mode(g, work);
        if constexpr (SHAPE == 128)
            if (far == 2) {
                CB_CLX(2);
                return;
            }
        if constexpr (SHAPE >= 128)
            if (far) {
                CB_CLX(1);
                return;
            }
        CB_CLX(0);
#undef CB_CLX
    });
}

}  // namespace

}  // namespace cb
