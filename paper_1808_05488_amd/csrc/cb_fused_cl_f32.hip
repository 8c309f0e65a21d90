// The channel-last fused kernel for float32 (cb_fused_cl.h) and the packing of its filter matrix.
#include "cb_fused_cl.h"

namespace cb {

namespace {

// Filter matrix of the float32 kernel: for every 16-row tile and k-group of 32, three fragments (terms h, m, l of the scaled value) of 64 x 16
// bytes: lane's 8 values are K(m = mtile*16 + lane%16, k' = kgroup*32 + 8*(lane/16) + 0..7), k' = (j*kw + i)*Cs + c; zero
// outside the filter matrix and for the channels c >= C of a padded pixel.
__global__ __launch_bounds__(256) void pack_fused_split_kernel(Geom g, int Mt16, int KG, const float* __restrict__ w,
                                                               uint4* __restrict__ KF)
{
    const long n = (long)Mt16 * KG * 64;
    const int taps = g.kh * g.kw;
    for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < n; e += (long)gridDim.x * 256) {
        const int lane = (int)(e & 63);
        const long gk = e >> 6;
        const int kgroup = (int)(gk % KG), mtile = (int)(gk / KG);
        const int m = mtile * 16 + (lane & 15);
        unsigned t[3][4];
#pragma unroll
        for (int q2 = 0; q2 < 4; ++q2) {
            float v[2];
#pragma unroll
            for (int o = 0; o < 2; ++o) {
                const int k = kgroup * 32 + 8 * (lane >> 4) + 2 * q2 + o;
                const int tap = k / g.Cs, c = k - tap * g.Cs;
                v[o] = (m < g.O && tap < taps && c < g.C) ? w[(size_t)m * g.R + (size_t)c * taps + tap] : 0.f;
            }
            split2(v[0], v[1], t[0][q2], t[1][q2], t[2][q2]);
        }
#pragma unroll
        for (int s = 0; s < 3; ++s) KF[(gk * 3 + s) * 64 + lane] = make_uint4(t[s][0], t[s][1], t[s][2], t[s][3]);
    }
}

}  // namespace

hipError_t launch_pack_fused_split(const Geom& g, const float* w, void* KF, hipStream_t st)
{
    const int KG = (g.Cs * g.kh * g.kw + 63) / 64 * 2, Mt16 = (g.O + 127) / 128 * 8;
    const long n = (long)Mt16 * KG * 64;
    unsigned grid = (unsigned)((n + 255) / 256);
    if (grid > 2048) grid = 2048;
    hipLaunchKernelGGL(pack_fused_split_kernel, dim3(grid), dim3(256), 0, st, g, Mt16, KG, w, (uint4*)KF);
    return hipGetLastError();
}

hipError_t launch_fused_f32_cl(const Geom& g, const FusedPlan& plan, const float* shadow, const int32_t* idx,
                               const int* count, const void* KF, const float* KT, const float* bias, int relu, float* OUT,
                               float* OUT2, const ClWork& work, hipStream_t st, Tm tm)
{
    return launch_fused_cl<float>(g, plan, shadow, idx, count, KF, KT, bias, relu, OUT, OUT2, work, st, tm);
}

}  // namespace cb
