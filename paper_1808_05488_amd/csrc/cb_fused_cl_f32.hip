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

// One row of the filter matrix a workgroup: the exponent of the power of two that takes its largest finite magnitude to 2^14 .. 2^15, and how many of its
// weights are, so scaled, below 2^-14 and not zero.
__global__ __launch_bounds__(256) void half_rows_kernel(Geom g, const float* __restrict__ w, int2* __restrict__ rows)
{
    __shared__ unsigned s_part[4];
    const int m = blockIdx.x, tid = threadIdx.x;
    auto reduce = [&](unsigned v, auto combine) {
        v = over_lanes<64>(v, combine);
        if ((tid & 63) == 0) s_part[tid >> 6] = v;
        __syncthreads();
        v = combine(combine(s_part[0], s_part[1]), combine(s_part[2], s_part[3]));
        __syncthreads();
        return v;
    };
    const float* const row = w + (size_t)m * g.R;
    const int R = m < g.O ? g.R : 0;
    unsigned most = 0u, lost = 0u;
    for (int k = tid; k < R; k += 256) {
        const unsigned b = __float_as_uint(row[k]) & 0x7FFFFFFFu;
        if (b < 0x7F800000u && b > most) most = b;
    }
    most = reduce(most, [](unsigned a, unsigned b) { return a > b ? a : b; });
    const int a = most ? 14 - ilogbf(__uint_as_float(most)) : 0;
    for (int k = tid; k < R; k += 256) lost += row[k] != 0.f && fabsf(ldexpf(row[k], a)) < 0x1p-14f ? 1u : 0u;
    lost = reduce(lost, [](unsigned a, unsigned b) { return a + b; });
    if (tid == 0) rows[m] = make_int2(a, (int)lost);
}

// The two float16 terms of the rows so scaled, in fragments like those of the three bfloat16 terms: h, and 2^11 times the rest.
__global__ __launch_bounds__(256) void pack_halves_kernel(Geom g, int Mt16, int KG, const float* __restrict__ w, const int2* __restrict__ rows, uint4* __restrict__ KH)
{
    const long n = (long)Mt16 * KG * 64;
    const int taps = g.kh * g.kw;
    for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < n; e += (long)gridDim.x * 256) {
        const int lane = (int)(e & 63);
        const long gk = e >> 6;
        const int kgroup = (int)(gk % KG), mtile = (int)(gk / KG);
        const int m = mtile * 16 + (lane & 15), a = rows[m].x;
        unsigned t[2][4];
#pragma unroll
        for (int q2 = 0; q2 < 4; ++q2) {
            float v[2];
#pragma unroll
            for (int o = 0; o < 2; ++o) {
                const int k = kgroup * 32 + 8 * (lane >> 4) + 2 * q2 + o;
                const int tap = k / g.Cs, c = k - tap * g.Cs;
                v[o] = (m < g.O && tap < taps && c < g.C) ? ldexpf(w[(size_t)m * g.R + (size_t)c * taps + tap], a) : 0.f;
            }
            halves2(v[0], v[1], 1.f, 2048.f, t[0][q2], t[1][q2]);
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) KH[(gk * 2 + s) * 64 + lane] = make_uint4(t[s][0], t[s][1], t[s][2], t[s][3]);
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
    if (cl_halves(g.O, ((unsigned)(g.Cs * g.kh * g.kw) + 31u) / 32u)) {
        uint4* const KH = (uint4*)KF + (size_t)n * 3;
        int2* const rows = (int2*)(KH + (size_t)n * 2);
        hipLaunchKernelGGL(half_rows_kernel, dim3((unsigned)Mt16 * 16u), dim3(256), 0, st, g, w, rows);
        hipLaunchKernelGGL(pack_halves_kernel, dim3(grid), dim3(256), 0, st, g, Mt16, KG, w, rows, KH);
    }
    return hipGetLastError();
}

hipError_t launch_fused_f32_cl(const Geom& g, const FusedPlan& plan, const float* shadow, const int32_t* idx,
                               const int* count, const void* KF, const float* KT, const float* bias, int relu, float* OUT,
                               float* OUT2, const ClWork& work, hipStream_t st, Tm tm)
{
    return launch_fused_cl<float>(g, plan, shadow, idx, count, KF, KT, bias, relu, OUT, OUT2, work, st, tm);
}

}  // namespace cb
