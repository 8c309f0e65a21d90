// Rules of the channel-last fused kernel (cb_fused_cl.hip) that need no GPU: plain arithmetic on the geometry, usable
// from host code and kernels alike.
#pragma once

#ifdef __HIPCC__
#define CB_HD __host__ __device__ __forceinline__
#else
#define CB_HD inline
#endif

namespace cb {

// Divisions by layer constants.  tap / kw = tap * inv_kw >> 16 for the few taps there are.  q / Wo = q * inv_wo >> 42
// with inv_wo = ceil(2^42 / Wo) (0: divide).  The quotient is exact while q * Wo < 2^42: q < 2^30 in every layer, so Wo < 2^12
// is enough.  The product lies below (q / Wo + 1) * 2^42 and has to fit 64 bits, which takes Ho <= 2^22.
struct ClDiv { unsigned long long inv_wo; unsigned inv_kw; };

inline ClDiv cl_div(int Wo, int Ho, int kw)
{
    ClDiv d;
    d.inv_wo = Wo < 4096 && Ho <= (1 << 22) ? ((1ull << 42) + (unsigned)Wo - 1ull) / (unsigned)Wo : 0ull;
    d.inv_kw = (65536u + (unsigned)kw - 1u) / (unsigned)kw;
    return d;
}

CB_HD int cl_row(const ClDiv& d, int q, int Wo) { return d.inv_wo ? (int)(((unsigned long long)(unsigned)q * d.inv_wo) >> 42) : q / Wo; }

}  // namespace cb
