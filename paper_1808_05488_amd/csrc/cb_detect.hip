// Change detection with closed-loop state update (Sec. III-A Eq. 3, Sec. III-C).
//
// HBM-bound streaming kernel: reads the frame and the input state once over all
// channels (2*C*P elements), writes a bit-packed change map (P/8 bytes) and
// copies the channels of changed pixels into the state.
//
// Mapping: a block of 256 threads is CS channel groups x PL pixel lanes
// (PL = 256/CS, a multiple of the 64-wide wavefront).  A lane owns VEC
// consecutive pixels (one 16-byte load per channel for float, VEC = 4) and its
// group walks the channels g, g+CS, ...; the per-group flags are OR-ed through
// LDS.  Splitting channels over groups multiplies the number of wavefronts in
// flight for layers with many channels and few pixels.
#include "cb_extract.h"
#include <algorithm>
#include <type_traits>

namespace cb {

namespace {

typedef unsigned uintx2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float widen(float v) { return v; }
__device__ __forceinline__ float widen(uint16_t v) { return __uint_as_float((uint32_t)v << 16); }

__device__ __forceinline__ float to_f(float v) { return v; }
__device__ __forceinline__ float to_f(uint16_t v) { return __uint_as_float((uint32_t)v << 16); }

template <typename T, int VEC> struct Pack;
template <> struct Pack<float, 4> { typedef float4 type; };
template <> struct Pack<float, 1> { typedef float type; };
template <> struct Pack<uint16_t, 4> { typedef uint2 type; };
template <> struct Pack<uint16_t, 1> { typedef uint16_t type; };

template <typename T, int VEC>
__device__ __forceinline__ void unpack(const typename Pack<T, VEC>::type& v, float (&f)[VEC]);
template <> __device__ __forceinline__ void unpack<float, 4>(const float4& v, float (&f)[4])
{ f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w; }
template <> __device__ __forceinline__ void unpack<float, 1>(const float& v, float (&f)[1]) { f[0] = v; }
template <> __device__ __forceinline__ void unpack<uint16_t, 4>(const uint2& v, float (&f)[4])
{
    f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xFFFF0000u);
    f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xFFFF0000u);
}
template <> __device__ __forceinline__ void unpack<uint16_t, 1>(const uint16_t& v, float (&f)[1])
{ f[0] = widen(v); }

// Load of a value that is used once (the new frame): marked non-temporal, so that it does not push
// the input state, which the next frame reads again, out of the caches.
template <typename V> __device__ __forceinline__ V ld_once(const V* p)
{
    typedef unsigned uvec __attribute__((ext_vector_type(sizeof(V) / 4 ? sizeof(V) / 4 : 1)));
    if constexpr (sizeof(V) >= 4) {
        const uvec u = __builtin_nontemporal_load(reinterpret_cast<const uvec*>(p));
        return __builtin_bit_cast(V, u);
    } else {
        return __builtin_nontemporal_load(p);
    }
}

// The VEC pixels of a channel at p.  bfloat16: at any alignment (a plane of an odd number of pixels leaves every other
// channel unaligned; global memory takes such loads, at the price of one more cache line per wavefront).
template <typename T, int VEC> struct PxMem { typedef typename Pack<T, VEC>::type type; };
typedef unsigned PxMem2x4 __attribute__((ext_vector_type(2), aligned(2)));
// (a type of its own for the loads that are not marked: of two loads of one type and address the compiler makes one, without the mark)
typedef unsigned long long PxMem64 __attribute__((aligned(2)));
template <> struct PxMem<uint16_t, 4> { typedef PxMem2x4 type; };
template <typename T, int VEC, bool ONCE> __device__ __forceinline__ typename Pack<T, VEC>::type ld_px(const T* p)
{
    typedef typename Pack<T, VEC>::type V;
    typedef typename PxMem<T, VEC>::type M;
    if constexpr (sizeof(T) == 2 && VEC > 1) {
        if constexpr (ONCE) return __builtin_bit_cast(V, (uintx2)__builtin_nontemporal_load(reinterpret_cast<const M*>(p)));
        else return __builtin_bit_cast(V, (unsigned long long)*reinterpret_cast<const PxMem64*>(p));
    } else {
        if constexpr (ONCE) return ld_once(reinterpret_cast<const V*>(p));
        else return *reinterpret_cast<const V*>(p);
    }
}
template <typename T, int VEC> __device__ __forceinline__ void st_px(T* p, const typename Pack<T, VEC>::type& v)
{
    typedef typename PxMem<T, VEC>::type M;
    if constexpr (sizeof(T) == 2 && VEC > 1) *reinterpret_cast<M*>(p) = __builtin_bit_cast(uintx2, v);
    else *reinterpret_cast<M*>(p) = v;
}

// Workgroup barrier that orders LDS accesses only.  __syncthreads() also waits until every global
// store of the wavefront has been acknowledged, which here would put one store latency on
// each round of the shadow update.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The value as the compiler cannot trace it back: what is computed from it stays where it is written.
__device__ __forceinline__ float opaque(float v) { asm volatile("" : "+v"(v)); return v; }
__device__ __forceinline__ uint16_t opaque(uint16_t v) { unsigned u = v; asm volatile("" : "+v"(u)); return (uint16_t)u; }

// bit i of a 16-bit value -> bit 4*i
__device__ __forceinline__ uint64_t spread4(uint64_t v)
{
    v = (v | (v << 24)) & 0x000000FF000000FFull;
    v = (v | (v << 12)) & 0x000F000F000F000Full;
    v = (v | (v << 6)) & 0x0303030303030303ull;
    v = (v | (v << 3)) & 0x1111111111111111ull;
    return v;
}

template <typename T, int VEC, int CS>
__global__ __launch_bounds__(256) void detect_kernel(const T* __restrict__ x, T* __restrict__ S, T* __restrict__ S2,
                                                     uint64_t* __restrict__ mbits0, int* __restrict__ ctl,
                                                     int C, int Cs, int P, int nwords, float tau, int flags)
{
    typedef typename Pack<T, VEC>::type V;
    const int par = ctl[CTL_FRAME] & 1;          // which of the two map buffers and counters this frame fills
    uint64_t* __restrict__ mbits = mbits0 + par;  // the two maps are interleaved: word w of this frame's map at [2 * w]
    int* __restrict__ nin = nin_counter(ctl, blockIdx.x, par);
    constexpr int PL = 256 / CS;
    constexpr unsigned ALL = (1u << VEC) - 1u;
    const int tid = threadIdx.x;
    const int g = tid / PL;
    const int pl = tid - g * PL;
    const long p0 = ((long)blockIdx.x * PL + pl) * VEC;
    const bool valid = p0 < P;

    unsigned bits = 0;
    if (valid && !(flags & DET_FORCE_ALL)) {
#pragma unroll 4
        for (int c = g; c < C; c += CS) {
            const size_t off = (size_t)c * P + p0;
            V xv = ld_once(reinterpret_cast<const V*>(x + off));
            V sv = *reinterpret_cast<const V*>(S + off);
            float xf[VEC], sf[VEC];
            unpack<T, VEC>(xv, xf);
            unpack<T, VEC>(sv, sf);
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                float d = xf[v] - sf[v];          // one float32 subtract, then |.| > tau (strict)
                bits |= (fabsf(d) > tau ? 1u : 0u) << v;
            }
        }
    }
    if (CS > 1) {
        __shared__ unsigned sflag[256];
        sflag[tid] = bits;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < CS; ++q) bits |= sflag[q * PL + pl];
    }
    if (flags & DET_FORCE_ALL) bits = valid ? ALL : 0u;

    // bit-packed change map, written by channel group 0
    if (g == 0) {
        const int lane = tid & 63;
        const long wave_p0 = ((long)blockIdx.x * PL + (pl & ~63)) * VEC;   // first pixel of this wavefront
        const long w0 = wave_p0 >> 6;
        if (VEC == 4) {
            uint64_t b0 = __ballot(bits & 1u), b1 = __ballot(bits & 2u);
            uint64_t b2 = __ballot(bits & 4u), b3 = __ballot(bits & 8u);
            if (lane < 4 && w0 + lane < nwords) {
                const int sh = 16 * lane;
                uint64_t w = spread4((b0 >> sh) & 0xFFFF) | (spread4((b1 >> sh) & 0xFFFF) << 1) |
                             (spread4((b2 >> sh) & 0xFFFF) << 2) | (spread4((b3 >> sh) & 0xFFFF) << 3);
                mbits[2 * (w0 + lane)] = w;
            }
            if (lane == 0) {
                int tot = __popcll(b0) + __popcll(b1) + __popcll(b2) + __popcll(b3);
                if (tot) atomicAdd(nin, tot);
            }
        } else {
            uint64_t b0 = __ballot(bits & 1u);
            if (lane == 0 && w0 < nwords) {
                mbits[2 * w0] = b0;
                int tot = __popcll(b0);
                if (tot) atomicAdd(nin, tot);
            }
        }
    }

    // state update: all channels of a changed pixel (closed loop), or every pixel
    unsigned upd = (flags & DET_NO_UPDATE) ? 0u : (flags & DET_COPY_ALL) ? (valid ? ALL : 0u) : bits;
    if (upd) {
        for (int c = g; c < C; c += CS) {
            const size_t off = (size_t)c * P + p0;
            if (upd == ALL) {
                *reinterpret_cast<V*>(S + off) = *reinterpret_cast<const V*>(x + off);
            } else {
#pragma unroll
                for (int v = 0; v < VEC; ++v)
                    if (upd & (1u << v)) S[off + v] = x[off + v];
            }
            if (S2) {
#pragma unroll
                for (int v = 0; v < VEC; ++v)
                    if (upd & (1u << v)) S2[(size_t)(p0 + v) * Cs + c] = x[off + v];
            }
        }
    }
}

// The LDS of a workgroup of the register-resident variant: flags of the channel groups, and for a shadow the staged pixels' numbers and rows.
template <typename T, int VEC, int CS, int CPT, int PLX, bool SH> struct DetectLds {
    static constexpr int PL = PLX ? PLX : (CS >= 4 ? 64 : 256 / CS), NT = PL * CS;
    static constexpr int EPV = 16 / (int)sizeof(T);  // elements per 16 bytes
    static constexpr int CMAX = CS * CPT;
    static constexpr int PITCH = CMAX + EPV;         // elements per staged pixel: 16-byte aligned rows, banks spread
    static constexpr int KMAX = NT * 16 / (PITCH * (int)sizeof(T)) > 0 ? NT * 16 / (PITCH * (int)sizeof(T)) : 1;
    static constexpr int flags = CS > 1 ? NT * 4 : 0, pix = SH ? PL * VEC * 4 : 0, rows = SH ? 2 * KMAX * PITCH * (int)sizeof(T) : 0;
    static constexpr int bytes = flags + pix + rows;
    static_assert(flags % 16 == 0 && pix % 16 == 0, "rows are 16-byte aligned");
};

// Arguments of detection with the extraction in the same launch
template <typename T> struct DetectArgs {
    const T* x;
    T *S, *S2;
    uint64_t* mbits0;
    int* ctl;
    int C, Cs;
    unsigned inv_per;
    int P, nwords;
    float tau;
    int flags;
    int2 stream;
    DetectJob job;
};

// Register-resident variant: a lane keeps the CPT channel values it compared, so
// the state update is stores only (no second, latency-bound read of the frame).
// Workgroup = CS channel groups x PL pixel lanes.
// PLX = 16 (one pixel per lane only): 16 instead of 64 pixel lanes per workgroup, for maps with so
// few pixels that 64-pixel workgroups would leave most compute units idle; such a workgroup owns a
// quarter of a 64-pixel word of the bit map and stores it as a half word.
// SH: the layer keeps a channel-last shadow of its state (S2), and channel q of group g is g*CPT + q instead of
// g + q*CS, so that a lane's channels are neighbours in the shadow.  C <= CS*CPT; the shadow's pixels are the C channels rounded
// up to whole 16-byte pieces, zero behind the last.  inv_per = ceil(2^20 / pieces of a pixel) divides a piece's number (below 1 024) by it.
// lds: detect_lds bytes (the extracting workgroups of the same launch put theirs to other uses).
// MAIL: the map also goes, tagged, to the extracting workgroups of the same launch (job), of which one that waits may have taken this block.  A block
// is what a workgroup, with one channel group a wavefront, detects.
template <typename T, int VEC, int CS, int CPT, int PLX, bool SH, bool MAIL>
__device__ __forceinline__
void detect_reg_block(const T* __restrict__ x, T* __restrict__ S, T* __restrict__ S2, uint64_t* __restrict__ mbits0,
                      int* __restrict__ ctl, int C, int Cs, unsigned inv_per, int P, int nwords, float tau, int flags, int2 stream, const DetectJob* job, unsigned bx, char* lds)
{
    typedef typename Pack<T, VEC>::type V;
    // which of the two map buffers and counters this frame fills: the frame count lives on the device
    // (the index extraction advances it), so that a captured launch replays correctly whatever the
    // number of frames captured
    const int frame = ctl[CTL_FRAME], par = frame & 1;
    const unsigned tag = (unsigned)frame + 1u;
    uint64_t* __restrict__ mbits = mbits0 + par;  // the two maps are interleaved: word w of this frame's map at [2 * w]
    int* __restrict__ nin = nin_counter(ctl, bx, par);
    constexpr int PL = PLX ? PLX : (CS >= 4 ? 64 : 256 / CS);
    static_assert(PLX == 0 || (PLX == 16 && VEC == 1 && CS > 1), "narrow workgroups: 16 lanes of one pixel each");
    constexpr int NT = PL * CS;
    constexpr unsigned ALL = (1u << VEC) - 1u;
    const int tid = threadIdx.x;
    const int g = tid / PL;
    const int pl = tid - g * PL;
    // The lane's pixels are pw .. pw + VEC - 1.  Where the image ends among them it loads the image's last VEC pixels
    // (p0 .. P - 1) instead, of which only those from pw on are its own.
    const long pw = ((long)bx * PL + pl) * VEC;
    const bool valid = pw < P;
    constexpr bool RAGGED = sizeof(T) == 2 && VEC > 1;      // (float32 takes several pixels per lane only where P is a multiple)
    const int over = RAGGED && valid && pw + VEC > P ? (int)(pw + VEC - P) : 0;
    const long p0 = pw - over;
    const unsigned own = valid ? (ALL << over) & ALL : 0u;

    // (stream: from and below which count of the frame before, still in place, the state is read once; float32 does not ask)
    bool once = (flags & DET_STREAM_STATE) != 0;
    if constexpr (sizeof(T) == 2)
        if (once) {
            const int before = __builtin_amdgcn_readfirstlane(ctl[CTL_COUNT]);
            once = before >= stream.x && before < stream.y;
        }

    const bool claimer = CS > 1 ? tid == 0 : (tid & 63) == 0;
    unsigned found = ~tag;                       // what the claim's word held
    // (behind the loads of the pixels, whose data it delays by nothing: results come in order.  Ahead of them, 0.5 us more in a frame of 43)
    auto claim = [&]() {
        if constexpr (MAIL)
            if (claimer) found = claim_block(DeviceMem(), job->claims + claim_index(CS > 1 ? bx : bx * (256 / 64) + (tid >> 6), (unsigned)job->nclaims), tag, &ctl[CTL_DONE], false);
    };

    uint64_t* const mail = MAIL ? job->mail : nullptr;

    V xv[CPT];
    unsigned bits = 0;
    if (valid) {
        if (flags & DET_FORCE_ALL) {
#pragma unroll
            for (int q = 0; q < CPT; ++q) {
                const int c = SH ? g * CPT + q : g + q * CS;
                if (c < C) xv[q] = ld_px<T, VEC, false>(x + (size_t)c * P + p0);
            }
            claim();
            // (first frame only.  Without this wait the compiler assumes these loads may still be in flight
            // in the other branch, and waits there between loads.)
            __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
        } else {
            V sv[CPT];
#pragma unroll
            for (int q = 0; q < CPT; ++q) {
                const int c = SH ? g * CPT + q : g + q * CS;
                if (c < C) {
                    const size_t off = (size_t)c * P + p0;
                    xv[q] = ld_px<T, VEC, true>(x + off);
                    sv[q] = once ? ld_px<T, VEC, true>(S + off) : ld_px<T, VEC, false>(S + off);
                }
            }
            claim();
            // every load is issued before the first compare waits for one: the kernel lives on loads in flight
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < CPT; ++q) {
                const int c = SH ? g * CPT + q : g + q * CS;
                if (c < C) {
                    float xf[VEC], sf[VEC];
                    unpack<T, VEC>(xv[q], xf);
                    unpack<T, VEC>(sv[q], sf);
#pragma unroll
                    for (int v = 0; v < VEC; ++v) {
                        float d = xf[v] - sf[v];      // one float32 subtract, then |.| > tau (strict)
                        bits |= (fabsf(d) > tau ? 1u : 0u) << v;
                    }
                }
            }
        }
    }
    if (CS > 1) {
        unsigned* const sflag = reinterpret_cast<unsigned*>(lds);
        constexpr unsigned LOST = 1u << 31;
        sflag[tid] = MAIL && tid == 0 && found == tag ? LOST : bits;
        __syncthreads();
        if (MAIL && sflag[0] == LOST) {
            if (tid == 0 && claim_lost(DeviceMem(), &ctl[CTL_DONE], job->nblk)) finish_frame(ctl, next_epoch((unsigned)ctl[CTL_EPOCH]), 1, false);
            return;
        }
#pragma unroll
        for (int q = 0; q < CS; ++q) bits |= sflag[q * PL + pl];
    } else if (MAIL && __builtin_amdgcn_readfirstlane(found) == tag) {
        if (claimer && claim_lost(DeviceMem(), &ctl[CTL_DONE], job->nblk)) finish_frame(ctl, next_epoch((unsigned)ctl[CTL_EPOCH]), 1, false);
        return;
    }
    bits = (flags & DET_FORCE_ALL) ? own : bits & own;

    if (g == 0) {
        const int lane = tid & 63;
        const long wave_p0 = ((long)bx * PL + (pl & ~63)) * VEC;
        const long w0 = wave_p0 >> 6;
        const unsigned mapped = bits >> over;
        if (VEC == 4) {
            uint64_t b0 = __ballot(mapped & 1u), b1 = __ballot(mapped & 2u);
            uint64_t b2 = __ballot(mapped & 4u), b3 = __ballot(mapped & 8u);
            if (lane < 4 && w0 + lane < nwords) {
                const int sh = 16 * lane;
                uint64_t w = spread4((b0 >> sh) & 0xFFFF) | (spread4((b1 >> sh) & 0xFFFF) << 1) |
                             (spread4((b2 >> sh) & 0xFFFF) << 2) | (spread4((b3 >> sh) & 0xFFFF) << 3);
                if constexpr (MAIL) {
                    mail_put(mail, 2 * (w0 + lane), tag, (unsigned)w);
                    mail_put(mail, 2 * (w0 + lane) + 1, tag, (unsigned)(w >> 32));
                }
                mbits[2 * (w0 + lane)] = w;
            }
            if (lane == 0) {
                int tot = __popcll(b0) + __popcll(b1) + __popcll(b2) + __popcll(b3);
                if (tot) atomicAdd(nin, tot);
            }
        } else if (PLX == 16) {
            // the active lanes are lanes 0-15 of the first wavefront: 16 consecutive pixels
            const unsigned b0 = (unsigned)__ballot(bits & 1u) & 0xFFFFu;
            if (lane == 0) {
                if constexpr (MAIL) {
                    mail_put(mail, bx, tag, b0);
                    // (the last word's units behind the image have no workgroup of their own)
                    if ((long)(bx + 1) * 16 >= P)
                        for (long u = (long)bx + 1; u < 4L * nwords; ++u) mail_put(mail, u, tag, 0u);
                }
                reinterpret_cast<uint16_t*>(mbits + 2 * (bx >> 2))[bx & 3] = (uint16_t)b0;
                if (b0) atomicAdd(nin, __popc(b0));
            }
        } else {
            uint64_t b0 = __ballot(bits & 1u);
            if (MAIL && lane < 2 && w0 < nwords) mail_put(mail, 2 * w0 + lane, tag, (unsigned)(b0 >> (32 * lane)));
            if (lane == 0 && w0 < nwords) {
                mbits[2 * w0] = b0;
                int tot = __popcll(b0);
                if (tot) atomicAdd(nin, tot);
            }
        }
    }

    unsigned upd = (flags & DET_NO_UPDATE) ? 0u : (flags & DET_COPY_ALL) ? own : bits;
    if (upd) {
#pragma unroll
        for (int q = 0; q < CPT; ++q) {
            const int c = SH ? g * CPT + q : g + q * CS;
            if (c < C) {
                const size_t off = (size_t)c * P + p0;
                const T* xe = reinterpret_cast<const T*>(&xv[q]);
                if (upd == ALL) {
                    st_px<T, VEC>(S + off, xv[q]);
                } else {
#pragma unroll
                    for (int v = 0; v < VEC; ++v)
                        if (upd & (1u << v)) S[off + v] = xe[v];
                }
            }
        }
    }

    // Shadow of a first layer: its few channels are in this lane's registers, a pixel is one 16-byte store (5 - 8 float32 channels: two).
    if constexpr (CS == 1) {
        if (S2 != nullptr && upd) {
            constexpr int EPV = 16 / (int)sizeof(T), PIECES = (CPT + EPV - 1) / EPV;
#pragma unroll
            for (int v = 0; v < VEC; ++v)
                if (upd & (1u << v)) {
#pragma unroll
                    for (int h = 0; h < PIECES; ++h) {
                        if (h * EPV >= Cs) break;
                        __attribute__((aligned(16))) T e[EPV];
#pragma unroll
                        for (int j = 0; j < EPV; ++j) {
                            const int c = h * EPV + j;
                            e[j] = c < CPT && c < C ? reinterpret_cast<const T*>(&xv[c < CPT ? c : 0])[v] : (T)0;
                        }
                        *reinterpret_cast<uint4*>(S2 + (size_t)(p0 + v) * Cs + h * EPV) = *reinterpret_cast<const uint4*>(e);
                    }
                }
        }
    }

    // Channel-last shadow of the state (pixel-major: the C values of a pixel side by side), kept for
    // the gather of the fused back end.  The values of a changed pixel sit in CS different lanes of
    // CS different wavefronts.  The changed pixels of the workgroup are numbered (lane-major, from
    // ballots: upd is the same in every channel group, so every wavefront finds the same numbers),
    // their values are staged in LDS, KMAX pixels at a time in two alternating buffers (one
    // barrier per round; 16 bytes per store: a lane's channels are neighbours), and written out as
    // whole rows, 16 bytes per thread.  The phase is kept short in instructions: a workgroup that
    // lingers here has no loads in flight, and the kernel lives on loads in flight.
    if constexpr (SH) {
        static_assert(CS >= 4 && (CPT * sizeof(T)) % 16 == 0, "shadow rows are staged 16 bytes at a time");
        if (S2 != nullptr) {
            typedef DetectLds<T, VEC, CS, CPT, PLX, SH> LDS;
            constexpr int EPV = LDS::EPV, CMAX = LDS::CMAX, PITCH = LDS::PITCH, KMAX = LDS::KMAX;
            int* const s_pix = reinterpret_cast<int*>(lds + LDS::flags);
            T (* const stage)[KMAX * PITCH] = reinterpret_cast<T (*)[KMAX * PITCH]>(lds + LDS::flags + LDS::pix);
            // a channel group is a whole wavefront, or (16-lane groups) a quarter of one
            const int lane = tid & 63;
            const int seg_shift = PL >= 64 ? 0 : (lane & ~(PL - 1));
            const uint64_t seg_mask = PL >= 64 ? ~0ull : ((1ull << (PL & 63)) - 1ull);
            const uint64_t below = (1ull << (lane & (PL >= 64 ? 63 : PL - 1))) - 1ull;
            int before = 0, total = 0;
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                const uint64_t bv = (__ballot((upd >> v) & 1u) >> seg_shift) & seg_mask;
                before += __popcll(bv & below);
                total += __popcll(bv);
            }
            if (g == 0) {
#pragma unroll
                for (int v = 0; v < VEC; ++v)
                    if (upd & (1u << v)) s_pix[before + __popc(upd & ((1u << v) - 1u))] = (int)(p0 + v);
            }
            const int per = Cs / EPV;                 // 16-byte pieces per pixel
            // bytes of a pixel's last piece that hold channels
            unsigned keep[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int n = (C - (Cs - EPV)) * (int)sizeof(T) - 4 * j;
                keep[j] = n >= 4 ? ~0u : n == 2 ? 0xFFFFu : 0u;
            }
            static_assert(KMAX * (CMAX / EPV) <= 1024, "pieces of a round, as inv_per takes them");
            // The 16-byte LDS stores want the same pixel of EPV channels in neighbouring registers,
            // the loads delivered the VEC pixels of one channel there.  Made opaque here, the
            // values are rearranged here -- and not right behind each load, where the compiler
            // would otherwise put the moves, with a wait for every single load in front of them.
            T xs[CPT][VEC];
#pragma unroll
            for (int q = 0; q < CPT; ++q)
#pragma unroll
                for (int v = 0; v < VEC; ++v) xs[q][v] = opaque(reinterpret_cast<const T*>(&xv[q])[v]);
            int buf = 0;
            for (int k0 = 0; k0 < total; k0 += KMAX, buf ^= 1) {
#pragma unroll
                for (int v = 0; v < VEC; ++v)
                    if (upd & (1u << v)) {
                        const int k = before + __popc(upd & ((1u << v) - 1u)) - k0;
                        if ((unsigned)k < (unsigned)KMAX) {
#pragma unroll
                            for (int q0 = 0; q0 < CPT; q0 += EPV) {
                                __attribute__((aligned(16))) T e[EPV];
#pragma unroll
                                for (int j = 0; j < EPV; ++j) e[j] = xs[q0 + j][v];
                                *reinterpret_cast<uint4*>(&stage[buf][k * PITCH + g * CPT + q0]) = *reinterpret_cast<const uint4*>(e);
                            }
                        }
                    }
                lds_barrier();                    // (also: s_pix is written; the buffer's readers of two rounds ago are done)
                const int nrow = total - k0 < KMAX ? total - k0 : KMAX;
                for (int i = tid; i < nrow * per; i += NT) {
                    const int k = (int)(((unsigned)i * inv_per) >> 20), pc = i - k * per;
                    typedef unsigned uvec4 __attribute__((ext_vector_type(4)));
                    uvec4 v4 = *reinterpret_cast<const uvec4*>(&stage[buf][k * PITCH + pc * EPV]);
                    if (pc == per - 1) v4 &= uvec4{keep[0], keep[1], keep[2], keep[3]};
                    __builtin_nontemporal_store(v4, reinterpret_cast<uvec4*>(S2 + (size_t)s_pix[k0 + k] * Cs + pc * EPV));
                }
            }
        }
    }
}

// A block of PX pixels in place of its own workgroup, which has not begun: a lane a pixel, channel by channel.  For launches that do not get the chip, and
// written to take no more registers than the rest.
template <typename T, int PX, int NT>
__device__ __forceinline__ void detect_taken(const T* __restrict__ x, T* S, T* S2, uint64_t* __restrict__ mbits0, int* __restrict__ ctl, int C, int Cs, int P, float tau,
                                             int flags, int b, int par, unsigned tag, uint64_t* mail)
{
    const int lane = threadIdx.x & 63;
    for (int o = threadIdx.x & ~63; o < PX; o += NT) {               // (whole wavefronts)
        const long p = (long)b * PX + o + lane;
        const bool valid = o + lane < PX && p < P;
        bool fired = valid && (flags & DET_FORCE_ALL);
#pragma unroll 1
        for (int c = 0; c < C && valid && !fired; ++c)
            fired = fabsf(widen(x[(size_t)c * P + p]) - widen(S[(size_t)c * P + p])) > tau;      // one float32 subtract, then |.| > tau (strict)
        const uint64_t word = __ballot(fired);
        if (valid && !(flags & DET_NO_UPDATE) && (fired || (flags & DET_COPY_ALL)))
#pragma unroll 1
            for (int c = 0; c < C; ++c) {
                S[(size_t)c * P + p] = x[(size_t)c * P + p];
                if (S2) S2[(size_t)p * Cs + c] = x[(size_t)c * P + p];
            }
        if (lane == 0) {
            const int n = __popcll(word);
            if (n) atomicAdd(nin_counter(ctl, (unsigned)b, par), n);
            const long w = (p >> 6);
            if (PX == 16) {
                reinterpret_cast<uint16_t*>(mbits0 + par + 2 * w)[b & 3] = (uint16_t)word;
                mail_put(mail, b, tag, (unsigned)word & 0xFFFFu);
                if ((long)(b + 1) * 16 >= P)
                    for (long u = (long)b + 1; u < 4L * ((P + 63) / 64); ++u) mail_put(mail, u, tag, 0u);
            } else if (p < P) {
                mbits0[2 * w + par] = word;
                mail_put(mail, 2 * w, tag, (unsigned)word);
                mail_put(mail, 2 * w + 1, tag, (unsigned)(word >> 32));
            }
        }
    }
}

template <typename T, int VEC, int CS, int CPT, int PLX = 0, bool SH = false>
__global__ __launch_bounds__((PLX ? PLX : (CS >= 4 ? 64 : 256 / CS)) * CS)
void detect_reg_kernel(const T* __restrict__ x, T* __restrict__ S, T* __restrict__ S2, uint64_t* __restrict__ mbits0,
                       int* __restrict__ ctl, int C, int Cs, unsigned inv_per, int P, int nwords, float tau, int flags, int2 stream)
{
    typedef DetectLds<T, VEC, CS, CPT, PLX, SH> LDS;
    __shared__ __align__(16) char lds[LDS::bytes ? LDS::bytes : 16];
    detect_reg_block<T, VEC, CS, CPT, PLX, SH, false>(x, S, S2, mbits0, ctl, C, Cs, inv_per, P, nwords, tau, flags, stream, nullptr, blockIdx.x, lds);
}

// Detection with the index extraction in the same launch: the last job.nblk workgroups extract (cb_claim.h).  A launch of its own costs the extraction
// 4 - 8 us, of which most is the end of one kernel, the start of the next and its first loads from memory.  Frames, us, two launches / one:
// 3 -> 16 at 48x64 14.4 / 11.1, 64 -> 64 at 480x640 43.0 / 42.0, 64 -> 128 at 271x435 bfloat16 25.8 / 22.0, 3 -> 16 7x7 at 1080p 33.7 / 30.8, feed-forward
// 64 -> 64 at 240x320 29.0 / 26.6.  (Without claims, whose answer a workgroup waits for: 11.0, 41.1, 21.5, 30.6, 26.4.)
template <typename T, int VEC, int CS, int CPT, int PLX = 0, bool SH = false>
__global__ __launch_bounds__((PLX ? PLX : (CS >= 4 ? 64 : 256 / CS)) * CS)
void detect_extract_kernel(const DetectArgs<T> a)
{
    constexpr int NT = (PLX ? PLX : (CS >= 4 ? 64 : 256 / CS)) * CS, PX = PLX ? PLX : 64 * VEC;      // (pixels of a block)
    typedef DetectLds<T, VEC, CS, CPT, PLX, SH> LDS;
    constexpr int EX = (MAP_STAGE * 8 + one_pass_small<NT / 64>() * 4 + 15) / 16 * 16, USED = LDS::bytes > EX ? LDS::bytes : EX;
    __shared__ __align__(16) char lds[USED + 16];
    unsigned* const s_word = reinterpret_cast<unsigned*>(lds + USED);            // (behind both uses of the LDS)
    const DetectJob& job = a.job;
    const Role role = role_of(job);
    int bid = 0;
    unsigned epoch = 0;
    detect_or_extract(
        role.extracts,
        [&]() {
            detect_reg_block<T, VEC, CS, CPT, PLX, SH, true>(a.x, a.S, a.S2, a.mbits0, a.ctl, a.C, a.Cs, a.inv_per, a.P, a.nwords, a.tau, a.flags, a.stream, &job, (unsigned)role.own, lds);
        },
        [&](bool limited) {
            const int frame = a.ctl[CTL_FRAME];
            if (limited) {
                bid = begin_extraction(a.ctl, job.nblk, s_word);
                if (threadIdx.x == 0) epoch = (unsigned)a.ctl[CTL_EPOCH];
                clear_other_map(a.mbits0, a.ctl, frame & 1, job.clear_words, bid * NT + (int)threadIdx.x, job.nblk * NT);
            }
            int polls = job.patience;
            return stage_own_block<NT>(job, bid, reinterpret_cast<uint64_t*>(lds), s_word, [&](long i, long step, long nw, uint64_t (&w)[2]) {
                return mail_words<PLX ? 64 / (PLX ? PLX : 1) : 2>(job.mail, i, step, nw, (unsigned)frame + 1u, w, limited, polls);
            });
        },
        [&]() {
            const DetectArgs<T> r = launch_arguments<DetectArgs<T>>();
            return unclaimed_block<NT>(r.job, r.job.nclaims, (unsigned)r.ctl[CTL_FRAME] + 1u, bid, reinterpret_cast<int*>(s_word));
        },
        [&](int b) {
            const DetectArgs<T> r = launch_arguments<DetectArgs<T>>();
            const int frame = r.ctl[CTL_FRAME];
            if (take_block(r.job, r.ctl, b, (unsigned)frame + 1u, s_word))
                detect_taken<T, PX, NT>(r.x, r.S, r.S2, r.mbits0, r.ctl, r.C, r.Cs, r.P, r.tau, r.flags, b, frame & 1, (unsigned)frame + 1u, r.job.mail);
        },
        [&]() {
            extract_own_block<NT>(job, a.ctl, bid, reinterpret_cast<const uint64_t*>(lds), epoch, reinterpret_cast<unsigned*>(lds + MAP_STAGE * 8), false);
        });
}

// State update as a kernel of its own, for frames whose change detection ran with DET_NO_UPDATE: all
// channels of every pixel that the change map marks are copied from the frame into the state (Sec. III-C)
// and, where the layer keeps one, into the channel-last shadow.  For states beyond the last-level
// cache, where the update inside the detection kernel costs far more than its bytes (a workgroup that
// stores anything leaves its compute unit without loads in flight): detection then is a pure
// stream, and this kernel touches the changed pixels only.
// A workgroup takes one 64-pixel word of the map at a time.  Phase 1, lane = pixel: the marked
// pixels' values of one channel go from the frame to the state (runs of pixels: part of a line)
// and into an LDS tile [changed pixel][channel]; phase 2, lane = channel: the tile's rows go to
// the shadow as contiguous pieces.  Channels in chunks of APPLY_CC.
constexpr int APPLY_CC = 128;
template <typename T>
__global__ __launch_bounds__(256) void state_apply_kernel(const T* __restrict__ x, T* __restrict__ S, T* __restrict__ S2,
                                                          const uint64_t* __restrict__ mbits0,
                                                          const int* __restrict__ ctl, int C, int Cs, int P, int nwords)
{
    typedef typename Pack<T, 4>::type V4;                  // four consecutive pixels of one channel
    constexpr int E16 = 16 / (int)sizeof(T);               // elements per 16 bytes
    constexpr int PITCH = APPLY_CC + E16;                  // 16-byte aligned rows, banks spread
    __shared__ __align__(16) T stage[64 * PITCH];
    __shared__ int s_pix[64];
    const int tid = threadIdx.x;
    const int quad = tid & 15, cg = tid >> 4;              // 16 groups of four pixels x 16 channel groups
    const int par = ctl[CTL_FRAME] & 1;                    // (the index extraction, which advances it, runs later)
    // groups of four pixels are 16-byte (8-byte) aligned in the frame and in the state
    const bool vec_ok = (P & 3) == 0 && (((uintptr_t)x | (uintptr_t)S) & (4 * sizeof(T) - 1)) == 0;
    for (int w = blockIdx.x; w < nwords; w += gridDim.x) {
        const uint64_t word = mbits0[2 * (long)w + par];
        if (word == 0) continue;                           // (uniform over the workgroup)
        const unsigned nib = (unsigned)(word >> (4 * quad)) & 15u;          // this thread's four pixels
        const int k0 = __popcll(word & ((1ull << (4 * quad)) - 1ull));       // changed pixels before them
        const int nchg = __popcll(word);
        const long p0 = (long)w * 64 + 4 * quad;
        if (cg == 0 && nib) {
            int k = k0;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (nib & (1u << j)) s_pix[k++] = (int)(p0 + j);
        }
        for (int c0 = 0; c0 < C; c0 += APPLY_CC) {
            const int cn = C - c0 < APPLY_CC ? C - c0 : APPLY_CC;
            if (nib) {
                // eight channels at a time: eight loads in flight, then their stores
                for (int cb = cg; cb < cn; cb += 128) {
                    T v[8][4];
                    if (nib == 15u && vec_ok) {
#pragma unroll
                        for (int i = 0; i < 8; ++i)
                            if (cb + 16 * i < cn) {
                                const V4 t4 = ld_once(reinterpret_cast<const V4*>(x + (size_t)(c0 + cb + 16 * i) * P + p0));
                                const T* e = reinterpret_cast<const T*>(&t4);
#pragma unroll
                                for (int j = 0; j < 4; ++j) v[i][j] = e[j];
                            }
#pragma unroll
                        for (int i = 0; i < 8; ++i)
                            if (cb + 16 * i < cn) {
                                V4 t4;
                                T* e = reinterpret_cast<T*>(&t4);
#pragma unroll
                                for (int j = 0; j < 4; ++j) e[j] = v[i][j];
                                *reinterpret_cast<V4*>(S + (size_t)(c0 + cb + 16 * i) * P + p0) = t4;
                            }
                    } else {
#pragma unroll
                        for (int i = 0; i < 8; ++i)
                            if (cb + 16 * i < cn) {
#pragma unroll
                                for (int j = 0; j < 4; ++j)
                                    if (nib & (1u << j)) v[i][j] = x[(size_t)(c0 + cb + 16 * i) * P + p0 + j];
                            }
#pragma unroll
                        for (int i = 0; i < 8; ++i)
                            if (cb + 16 * i < cn) {
#pragma unroll
                                for (int j = 0; j < 4; ++j)
                                    if (nib & (1u << j)) S[(size_t)(c0 + cb + 16 * i) * P + p0 + j] = v[i][j];
                            }
                    }
                    if (S2) {
#pragma unroll
                        for (int i = 0; i < 8; ++i)
                            if (cb + 16 * i < cn) {
                                int k = k0;
#pragma unroll
                                for (int j = 0; j < 4; ++j)
                                    if (nib & (1u << j)) stage[(k++) * PITCH + cb + 16 * i] = v[i][j];
                            }
                    }
                }
            }
            if (S2) {
                const int cs = Cs - c0 < APPLY_CC ? Cs - c0 : APPLY_CC, zero = cs - cn;     // channels that pad a pixel of the shadow: up to 3 / 7
                for (int i = tid; i < nchg * zero; i += 256) stage[(i / zero) * PITCH + cn + i % zero] = (T)0;
                __syncthreads();
                const int per = cs / E16;                  // 16-byte pieces per pixel
                for (int i = tid; i < nchg * per; i += 256) {
                    const int kk = i / per, pc = i - kk * per;
                    typedef unsigned uvec4 __attribute__((ext_vector_type(4)));
                    const uvec4 v4 = *reinterpret_cast<const uvec4*>(&stage[kk * PITCH + pc * E16]);
                    __builtin_nontemporal_store(v4, reinterpret_cast<uvec4*>(S2 + (size_t)s_pix[kk] * Cs + c0 + pc * E16));
                }
                __syncthreads();                           // the tile and s_pix are rewritten by the next chunk / word
            }
        }
    }
}

// The whole shadow from the state: S (C x P) -> S2 (P x C), 64 x 64 tiles through LDS.  For a state that
// arrives from outside (an imported checkpoint); not on the per-frame path.
template <typename T>
__global__ __launch_bounds__(256) void shadow_rebuild_kernel(const T* __restrict__ S, T* __restrict__ S2, int C, int Cs, int P)
{
    __shared__ T tile[64][65];
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const int ctiles = (C + 63) / 64;
    const long tiles = (((long)P + 63) / 64) * ctiles;
    for (long t = blockIdx.x; t < tiles; t += gridDim.x) {
        const long pt = t / ctiles;
        const int c0 = (int)(t - pt * ctiles) * 64;
        const long p0 = pt * 64;
        for (int r = ty; r < 64; r += 4)                   // row = channel, lane = pixel
            if (c0 + r < C && p0 + tx < P) tile[r][tx] = S[(size_t)(c0 + r) * P + p0 + tx];
        __syncthreads();
        for (int r = ty; r < 64; r += 4)                   // row = pixel, lane = channel
            if (c0 + tx < C && p0 + r < P) S2[(size_t)(p0 + r) * Cs + c0 + tx] = tile[tx][r];
        __syncthreads();
    }
}

// The extraction inside the launch of detection, by workgroups of nt threads: words of the dilated map per wavefront (0: it takes a launch
// of its own).  The part of the map under one workgroup's words fits its LDS, and the workgroups that wait are at most a quarter of a whole chip's wavefronts: what
// they wait for runs beside them (that it is ever done does not depend on that, cb_claim.h).  Few words a wavefront spread the expansion of dense words and shorten the polls, many workgroups add up more
// counts and poll for more of each other's rows.  Frames, us (without claims), 16 / 32 / 64 words: 3 -> 16, 7x7, 1080p (507, 254, 127 workgroups) 36.3 / 32.0 / 30.4;
// 3 -> 16 at 720p (225, 113, 57) 18.2 / 16.8 / 16.9; 3 -> 16 at 240x320 (19, 10, 5) 13.1 / 13.4 / 14.1; 64 -> 32 at 120x160 14.8 / 15.0 / 15.9; 64 -> 64 at
// 480x640, 20 % (38, 19, 10) 81.5 / 82.2 / 84.8; 128 -> 64 at 46x82, bfloat16 (2, 1, 1) 16.4 / 15.6 / 16.1.
// Where one workgroup has them all in any case, 16 a wavefront occupy more of its wavefronts (16 / 32 words): 3 -> 16 at 48x64, 30 % changed, 11.1 / 11.9, 64 -> 64 at 40x60
// 12.5 / 13.1, 16 -> 16 5x5 at 60x60 11.5 / 12.2, five-layer net at 100x128 87.0 / 89.4.
int extract_words(const Geom& g, int nt)
{
    if (g.s > 2) return 0;
    const long items = (long)g.Ho * g.WWo;
    auto blocks = [&](int per) { return (items - 1) / (nt / 64 * per) + 1; };
    const int per = blocks(16) == 1 || (blocks(16) > 2 && blocks(16) <= 40) ? 16 : blocks(32) <= 80 ? 32 : 64;
    const long ipb = nt / 64 * per;
    const long rows = std::min<long>((ipb - 1 + g.WWo - 1) / g.WWo * g.s + std::max(g.kh, g.s) + 1 + g.p, g.H);
    return blocks(per) * nt <= 131072 && rows * g.W / 64 + 5 <= MAP_STAGE ? per : 0;
}

template <typename T, int VEC, int CS, int CPT, int PLX = 0>
void launch_reg(const T* x, T* S, T* S2, uint64_t* mbits, int* ctl, int C, int Cs, int P, float tau, int flags, int2 stream, DetectJob* job, hipStream_t st, Tm tm)
{
    constexpr int PL = PLX ? PLX : (CS >= 4 ? 64 : 256 / CS);
    const long px_per_block = (long)PL * VEC;
    const unsigned grid = (unsigned)((P + px_per_block - 1) / px_per_block);
    const unsigned per = (unsigned)Cs * (unsigned)sizeof(T) / 16u, inv_per = per ? ((1u << 20) + per - 1u) / per : 0u;
    // (job->nblk stays 0 where the extraction takes a launch of its own)
    // A workgroup of 16 wavefronts with eight bfloat16 channels a lane has little to load and one other beside it on its compute unit, so that the answer of a claim, waited for by
    // all of it, is not hidden: from more workgroups on than run at once (512) every round of them pays it.  Frames, us, in one launch / a launch of its own, 0.3 and 10 % changed: 128 -> 64 at
    // 1080p 208.7 / 183.7 and 381.4 / 358.2, at 720x1280 91.9 / 78.2 and 165.8 / 152.4, at 480x640 40.8 / 37.2 and 60.5 / 56.9; 80 -> 128 at 600x800 44.8 / 37.1 and 72.2 / 65.3; 96 -> 64 at
    // 360x640 (900 workgroups) 29.3 / 27.3 and 42.5 / 40.8; 128 -> 128 at 1080p 213.3 / 185.8 and 458.3 / 460.2 (as a first frame 442 / 421); one round: 128 -> 64 at 270x480 (507) 22.7 / 22.5 and 31.4 / 32.9.
    const bool alone = sizeof(T) == 2 && VEC == 4 && CS == 16 && CPT == 8 && grid > 512u;
    if (job && (job->per = alone ? 0 : extract_words(job->g, PL * CS)) > 0) job->nblk = (job->g.Ho * job->g.WWo - 1) / (PL * CS / 64 * job->per) + 1;
    if (job) job->inv_wwo = map_row_inv((unsigned)job->g.WWo);
    if (job && job->ahead) job->ahead = job->nblk;
    if (job) job->nclaims = CS > 1 ? (int)grid : (P + 64 * VEC - 1) / (64 * VEC);
#define CB_REG(sh, shadow)                                                                                                          \
    if (job && job->nblk)                                                                                                           \
        CB_LAUNCH((detect_extract_kernel<T, VEC, CS, CPT, PLX, sh>), dim3(grid + (unsigned)job->nblk), dim3(PL * CS), st, tm,       \
                  (DetectArgs<T>{x, S, shadow, mbits, ctl, C, Cs, inv_per, P, (P + 63) / 64, tau, flags, stream, *job}));             \
    else CB_LAUNCH((detect_reg_kernel<T, VEC, CS, CPT, PLX, sh>), dim3(grid), dim3(PL * CS), st, tm, x, S, shadow, mbits, ctl, C, Cs, \
              inv_per, P, (P + 63) / 64, tau, flags, stream)
    if constexpr (CS >= 4 && (CPT * sizeof(T)) % 16 == 0) {
        // (launch_t only passes a shadow on when the variant's registers hold all C channels)
        if (S2 != nullptr) {
            CB_REG(true, S2);
            return;
        }
    }
    CB_REG(false, CS == 1 ? S2 : (T*)nullptr);
#undef CB_REG
}

template <typename T, int VEC>
void launch_v(const T* x, T* S, T* S2, uint64_t* mbits, int* ctl, int C, int Cs, int P, float tau, int flags, int2 stream, DetectJob* job, hipStream_t st, Tm tm)
{
    // channel groups CS and channels per lane CPT with CS*CPT >= C
    if (C <= 4)        launch_reg<T, VEC, 1, 4>(x, S, S2, mbits, ctl, C, Cs, P, tau, flags, stream, job, st, tm);
    else if (C <= 8)   launch_reg<T, VEC, 1, 8>(x, S, S2, mbits, ctl, C, Cs, P, tau, flags, stream, job, st, tm);
    // (bfloat16 with a shadow: eight channels per lane are one of its 16-byte pieces)
    else if (C <= 16 && !(sizeof(T) == 2 && S2)) launch_reg<T, VEC, 4, 4>(x, S, S2, mbits, ctl, C, Cs, P, tau, flags, stream, job, st, tm);
    else if (C <= 32)  launch_reg<T, VEC, 4, 8>(x, S, S2, mbits, ctl, C, Cs, P, tau, flags, stream, job, st, tm);
    else if (C <= 64)  launch_reg<T, VEC, 8, 8>(x, S, S2, mbits, ctl, C, Cs, P, tau, flags, stream, job, st, tm);
    // maps of fewer than 128 x 64 pixels with many channels: 16-pixel workgroups reach every compute unit
    else if (VEC == 1 && P < 8192 && C <= 128) launch_reg<T, 1, 16, 8, 16>(x, S, S2, mbits, ctl, C, Cs, P, tau, flags, stream, job, st, tm);
    else if (VEC == 1 && P < 8192 && C <= 256) launch_reg<T, 1, 16, 16, 16>(x, S, S2, mbits, ctl, C, Cs, P, tau, flags, stream, job, st, tm);
    else if (VEC == 1 && P < 8192 && C <= 512) launch_reg<T, 1, 16, 32, 16>(x, S, S2, mbits, ctl, C, Cs, P, tau, flags, stream, job, st, tm);
    else if (C <= 128) launch_reg<T, VEC, 16, 8>(x, S, S2, mbits, ctl, C, Cs, P, tau, flags, stream, job, st, tm);
    // (129 - 256 bfloat16 channels: 82 registers.  They walked their channels one by one, or 2 bytes per lane and load: frames, us,
    // 160 channels, 1x1, at 540x960 116 -> 77, 256 channels there 181 -> 105, at 180x200 36 -> 29.  float32 would need 140 registers.)
    else if (VEC == 4 && sizeof(T) == 2 && C <= 256) {
        if constexpr (VEC == 4 && sizeof(T) == 2) launch_reg<T, 4, 16, 16>(x, S, S2, mbits, ctl, C, Cs, P, tau, flags, stream, job, st, tm);
    }
    // one pixel per lane leaves registers for more channels per lane (deep layers: many channels, few pixels)
    else if (VEC == 1 && C <= 256) launch_reg<T, 1, 16, 16>(x, S, S2, mbits, ctl, C, Cs, P, tau, flags, stream, job, st, tm);
    else if (VEC == 1 && C <= 512) launch_reg<T, 1, 16, 32>(x, S, S2, mbits, ctl, C, Cs, P, tau, flags, stream, job, st, tm);
    else {
        // more channels than the register-resident variants hold: looped variant
        const long px_per_block = 64L * VEC;
        const unsigned grid = (unsigned)((P + px_per_block - 1) / px_per_block);
        CB_LAUNCH((detect_kernel<T, VEC, 4>), dim3(grid), dim3(256), st, tm, x, S, S2, mbits, ctl, C, Cs, P,
                  (P + 63) / 64, tau, flags);
    }
}

template <typename T> struct ListedArgs {
    const T* x;
    T *S, *S2;
    uint64_t* mbits0;
    int* ctl;
    const int32_t* cand;
    const int* cand_count;
    int cand_cap, C, Cpx, P, W;
    float tau;
    int flags, pool_w, cand_W, unused;
    DetectJob job;
};

// Change detection restricted to candidate pixels (Eq. 3 where it can fire at all).  When a
// layer's input is the cached output of a change-based producer, only the producer's listed
// pixels were rewritten; every other input pixel holds the bits it held a frame ago, when it
// did not fire against the same state, so it cannot fire now.  Lane = candidate n, CS channel
// groups per workgroup; a first pass compares all channels of the candidate (flags OR-ed
// through LDS), a second pass copies the pixel into the state where it fired.  Bits are set
// with atomic ORs into the (pre-cleared) linear bit map, one per run of candidates that share
// a word; the changed-pixel count adds the bits that were newly set, so a pixel reached through
// several candidates (2x2 pooling maps up to four of them to one pixel) is counted once.  Duplicates race benignly: whoever copies the
// pixel first makes the others compare equal, and the bit is set either way.
// SH: the layer keeps a channel-last shadow S2 of its state and C is a power of two (other shadows are written from registers).  The values of the candidates are
// staged in LDS ahead of the first barrier of a round and, once it is known which candidates fired, written to
// S2 with consecutive lanes on consecutive channels; two alternating buffers, so the barriers the round has anyway
// are enough.  (Written from the registers that hold them they are 4-byte stores to a different line per lane.)
constexpr int LISTED_U = 8, LISTED_BLOCKS = 2048;
template <typename T, int CS, int PLC, bool SH> struct ListedLds {
    static constexpr int PITCH = CS * LISTED_U + 1;   // staged values per candidate: candidates a lane apart fall into different banks
    // (one buffer and a barrier at the end of the round where two would not fit)
    static constexpr int NBUF = PLC * PITCH * (int)sizeof(T) * 2 <= 32768 ? 2 : 1;
    static constexpr int flags = CS * PLC * 4, rows = SH ? (NBUF * PLC * PITCH * (int)sizeof(T) + 15) / 16 * 16 : 0, pix = SH ? NBUF * PLC * 4 : 0;
    static constexpr int bytes = flags + rows + pix;
};
// Workgroup bx of `blocks`; lds: ListedLds bytes.  ARRIVE: it adds itself to the arrivals when its bits are set, and claims its block of the job first if it
// has pixels (a waiting workgroup may have taken it).
template <typename T, int CS, int PLC, bool SH, bool ARRIVE>
__device__ __forceinline__ void detect_listed_block(const T* __restrict__ x, T* __restrict__ S,
                                                    T* __restrict__ S2, uint64_t* __restrict__ mbits0,
                                                    int* __restrict__ ctl,
                                                    const int32_t* __restrict__ cand,
                                                    const int* __restrict__ cand_count, int cand_cap,
                                                    int C, int Cpx, int P, int W, float tau, int flags, int pool_w,
                                                    int cand_W, int bx, int blocks, const DetectJob* job, char* lds)
{
    constexpr int U = LISTED_U;                   // channels per lane held in registers (all of them when C <= 8*CS)
    const int frame = ctl[CTL_FRAME], par = frame & 1;          // which of the two map buffers and counters this frame fills
    uint64_t* __restrict__ mbits = mbits0 + par;  // the two maps are interleaved: word w of this frame's map at [2 * w]
    int* __restrict__ nin = nin_counter(ctl, (unsigned)bx, par);
    const unsigned tag = (unsigned)frame + 1u;
    unsigned found = ~tag;                        // (thread 0) what the claim's word held
    typedef ListedLds<T, CS, PLC, SH> LDS;
    unsigned* const sflag = reinterpret_cast<unsigned*>(lds);
    constexpr int PITCH = LDS::PITCH, NBUF = LDS::NBUF;
    T (* const stage)[SH ? PLC * PITCH : 1] = reinterpret_cast<T (*)[SH ? PLC * PITCH : 1]>(lds + LDS::flags);
    int (* const s_q)[SH ? PLC : 1] = reinterpret_cast<int (*)[SH ? PLC : 1]>(lds + LDS::flags + LDS::rows);
    const int tid = threadIdx.x, g = tid / PLC, pl = tid - g * PLC;
    const int Cs = C < CS * U ? C : CS * U;       // channels held in registers (SH: a power of two)
    const int lcs = 31 - __builtin_clz((unsigned)Cs);
    int buf = 0;
    // the candidate of the first round is requested together with the count (the list has cand_cap
    // entries; those beyond the count are stale but readable), later ones a round ahead
    const int step = blocks * PLC;
    int nnext = bx * PLC + pl;
    int qnext = cand[nnext < cand_cap ? nnext : cand_cap - 1];
    const int nc = *cand_count;
    for (int t0 = bx * PLC; t0 < nc; t0 += step) {
        const int n = t0 + pl;
        const bool valid = n < nc;
        int q = valid ? qnext : 0;
        nnext = n + step;
        qnext = cand[nnext < cand_cap ? nnext : cand_cap - 1];
        if (pool_w > 1) {
            const int yo = q / cand_W, xo = q - yo * cand_W;
            q = (yo / pool_w) * W + xo / pool_w;
        }
        unsigned fired = 0;
        T xr[U];
        if (ARRIVE && tid == 0 && t0 == bx * PLC) found = claim_block(DeviceMem(), job->claims + claim_index((unsigned)bx, (unsigned)job->nclaims), tag, &ctl[CTL_DONE], false);
        if (valid) {
            T sr[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {         // surplus loads repeat channel 0 (a layer may have fewer
                const int c = g + u * CS;         // channels than the workgroup has channel groups)
                const size_t off = (size_t)(c < C ? c : 0) * P + q;
                xr[u] = x[off];
                sr[u] = S[off];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float d = to_f(xr[u]) - to_f(sr[u]);   // one float32 subtract, then |.| > tau (strict)
                fired |= (fabsf(d) > tau) ? 1u : 0u;
            }
            for (int c = g + U * CS; c < C; c += CS) {       // more channels than the registers hold
                const size_t off = (size_t)c * P + q;
                const float d = to_f(x[off]) - to_f(S[off]);
                fired |= (fabsf(d) > tau) ? 1u : 0u;
            }
        }
        if (SH && valid) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int c = g + u * CS;
                if (c < C) stage[SH ? buf : 0][SH ? pl * PITCH + c : 0] = xr[u];
            }
        }
        constexpr unsigned LOST = 1u << 31;
        sflag[tid] = ARRIVE && tid == 0 && found == tag ? LOST : fired;
        __syncthreads();
        if (ARRIVE && sflag[0] == LOST) {
            if (tid == 0 && claim_lost(DeviceMem(), &ctl[CTL_DONE], job->nblk)) finish_frame(ctl, next_epoch((unsigned)ctl[CTL_EPOCH]), 1, true);
            return;
        }
#pragma unroll
        for (int k = 0; k < CS; ++k) fired |= sflag[k * PLC + pl];
        if (SH && g == 0) s_q[SH ? buf : 0][SH ? pl : 0] = (valid && (fired || (flags & DET_COPY_ALL))) ? q : -1;
        __syncthreads();                          // sflag is rewritten in the next round
        auto set_bits = [&]() {
            // The first wavefront (PLC lanes of it have a candidate).  Neighbouring candidates mostly fall into the same
            // 32-pixel word of the map: the bits of a word are combined and set with ONE atomic -- a
            // few thousand atomics on a few hundred words otherwise queue up behind each other.  (A word at a time with lane reads and data-parallel-primitive moves; a
            // segmented OR over all lanes takes a dozen shuffles, an LDS round trip each.)
            const int lane = tid & 63;
            const bool set = lane < PLC && valid && fired;
            const unsigned bit = set ? 1u << (q & 31) : 0u;
            const int word = q >> 5;
            uint64_t left = __ballot(set);
            unsigned bits = 0;                                // of the lane-th word
            int at = 0, words = 0;
            for (; left && words < 8; ++words) {
                const int w = __builtin_amdgcn_readlane(word, __builtin_ctzll(left));
                const bool here = set && word == w;
                left &= ~__ballot(here);
                const unsigned all = (unsigned)wave_or(here ? (int)bit : 0);
                if (lane == words) { bits = all; at = w; }
            }
            uint32_t* const map = reinterpret_cast<uint32_t*>(mbits);
            unsigned old = 0, alone = 0;
            if (lane < words) old = atomicOr(map + 4 * (at >> 1) + (at & 1), bits);
            const bool more = (left >> lane) & 1ull;          // (scattered over more words: a pixel each)
            if (more) alone = atomicOr(map + 4 * (word >> 1) + (word & 1), bit);
            if (ARRIVE && t0 + step >= nc && tid == 0) arrive(ctl, (unsigned)bx);
            // a pixel reached through several candidates counts once
            const int fresh = wave_sum(__popc(bits & ~old) + (more && !(alone & bit) ? 1 : 0));
            if (lane == 0 && fresh) atomicAdd(nin, fresh);
        };
        // State update first: it does not depend on the bit map.  Where extracting workgroups wait for the bits, these go first,
        // and the workgroup arrives as soon as its last are set (behind the state update it would wait for those stores too).
        if (ARRIVE && tid < 64) set_bits();
        if (valid && (fired || (flags & DET_COPY_ALL))) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int c = g + u * CS;
                if (c < C) {
                    S[(size_t)c * P + q] = xr[u];
                    if (!SH && S2) S2[(size_t)q * Cpx + c] = xr[u];
                }
            }
            for (int c = g + U * CS; c < C; c += CS) {
                const size_t off = (size_t)c * P + q;
                const T xc = x[off];
                S[off] = xc;
                if (S2) S2[(size_t)q * Cpx + c] = xc;
            }
        }
        if (SH) {
            // rows of the candidates that fired (buffer `buf`: the next round fills the other one)
            for (int i = tid; i < (PLC << lcs); i += CS * PLC) {
                const int row = i >> lcs, c = i & (Cs - 1);
                const int qq = s_q[SH ? buf : 0][SH ? row : 0];
                if (qq >= 0) S2[(size_t)qq * C + c] = stage[SH ? buf : 0][SH ? row * PITCH + c : 0];
            }
            if (NBUF == 2) buf ^= 1;
            else lds_barrier();
        }
        if (!ARRIVE && tid < 64) set_bits();
    }
}

// The candidates of workgroup bx in its place, as detect_taken: a wavefront a candidate, a lane a channel.
template <typename T, int PLC, int NT>
__device__ __forceinline__ void detect_listed_taken(const T* __restrict__ x, T* S, T* S2, uint64_t* __restrict__ mbits0, int* __restrict__ ctl, const int32_t* __restrict__ cand,
                                                    int nc, int C, int Cpx, int P, int W, float tau, int flags, int pool_w, int cand_W, int bx, int blocks, int par)
{
    const int lane = threadIdx.x & 63;
    int fresh = 0;
    for (int i = threadIdx.x >> 6;; i += NT / 64) {
        const long n = (long)(i / PLC * blocks + bx) * PLC + i % PLC;
        if (n - i % PLC >= nc) break;
        if (n >= nc) continue;
        int q = cand[n];
        if (pool_w > 1) {
            const int yo = q / cand_W, xo = q - yo * cand_W;
            q = (yo / pool_w) * W + xo / pool_w;
        }
        bool fired = false;
#pragma unroll 1
        for (int c = lane; c < C; c += 64) fired |= fabsf(to_f(x[(size_t)c * P + q]) - to_f(S[(size_t)c * P + q])) > tau;     // one float32 subtract, then |.| > tau (strict)
        fired = __ballot(fired) != 0;
        if (fired && lane == 0) {
            const unsigned bit = 1u << (q & 31);
            if (!(atomicOr(reinterpret_cast<uint32_t*>(mbits0 + par + 2 * (q >> 6)) + (q >> 5 & 1), bit) & bit)) ++fresh;
        }
        if (fired || (flags & DET_COPY_ALL))
#pragma unroll 1
            for (int c = lane; c < C; c += 64) {
                S[(size_t)c * P + q] = x[(size_t)c * P + q];
                if (S2) S2[(size_t)q * Cpx + c] = x[(size_t)c * P + q];
            }
    }
    if (fresh) atomicAdd(nin_counter(ctl, (unsigned)bx, par), fresh);
    __syncthreads();                              // (every bit's atomic has returned its old value)
    if (threadIdx.x == 0) arrive(ctl, (unsigned)bx);
}

template <typename T, int CS, int PLC, bool SH = false>
__global__ __launch_bounds__(CS * PLC) void detect_listed_kernel(const T* __restrict__ x, T* __restrict__ S,
                                                                 T* __restrict__ S2, uint64_t* __restrict__ mbits0,
                                                                 int* __restrict__ ctl,
                                                                 const int32_t* __restrict__ cand,
                                                                 const int* __restrict__ cand_count, int cand_cap,
                                                                 int C, int Cpx, int P, int W, float tau, int flags, int pool_w,
                                                                 int cand_W)
{
    __shared__ __align__(16) char lds[ListedLds<T, CS, PLC, SH>::bytes];
    detect_listed_block<T, CS, PLC, SH, false>(x, S, S2, mbits0, ctl, cand, cand_count, cand_cap, C, Cpx, P, W, tau, flags, pool_w, cand_W, (int)blockIdx.x, (int)gridDim.x,
                                              nullptr, lds);
}

// Detection at listed pixels with the index extraction in the same launch, as detect_extract_kernel.  Frames, us, two launches a layer / one: five-layer 7 x 7 net
// at 480x640 with detection in every layer 144 / 130, bfloat16 117 / 104, ten-layer 3 x 3 trunk at 368x656 394 / 375, bfloat16 269 / 257, at
// 150x200 204.5 / 200.5.  (State update ahead of the bits, as in the launch by itself, gains half of that.  Extracting workgroups in front: the same within 0.5 %, but
// 355 instead of 346 on the bfloat16 trunk with 20 % of its pixels changed; 512 detecting workgroups at most 356 there.)
template <typename T, int CS, int PLC, bool SH = false>
__global__ __launch_bounds__(CS * PLC) void detect_listed_extract_kernel(const ListedArgs<T> a)
{
    constexpr int NT = CS * PLC, EX = (MAP_STAGE * 8 + one_pass_small<NT / 64>() * 4 + 15) / 16 * 16, LI = (ListedLds<T, CS, PLC, SH>::bytes + 15) / 16 * 16,
                  USED = EX > LI ? EX : LI;
    __shared__ __align__(16) char lds[USED + 16];
    unsigned* const s_word = reinterpret_cast<unsigned*>(lds + USED);
    const Role role = role_of(a.job);
    const int blocks = role.n;
    int bid = 0;
    auto busy = [&](const int* count) {
        const int want = (*count + PLC - 1) / PLC;
        return want < blocks ? want : blocks;
    };
    unsigned epoch = 0;
    detect_or_extract(
        role.extracts,
        [&]() {
            detect_listed_block<T, CS, PLC, SH, true>(a.x, a.S, a.S2, a.mbits0, a.ctl, a.cand, a.cand_count, a.cand_cap, a.C, a.Cpx, a.P, a.W, a.tau, a.flags, a.pool_w, a.cand_W,
                                                     role.own, blocks, &a.job, lds);
        },
        [&](bool limited) {
            const ListedArgs<T> r = launch_arguments<ListedArgs<T>>();
            const int par = r.ctl[CTL_FRAME] & 1;
            if (limited) {
                bid = begin_extraction(r.ctl, r.job.nblk, s_word);
                if (threadIdx.x == 0) epoch = (unsigned)r.ctl[CTL_EPOCH];
                clear_other_map(r.mbits0, r.ctl, par, r.job.clear_words, bid * NT + (int)threadIdx.x, r.job.nblk * NT);
            }
            return await_arrivals(r.ctl, busy(r.cand_count), limited, r.job.patience, s_word) &&
                   stage_own_block<NT>(r.job, bid, reinterpret_cast<uint64_t*>(lds), s_word,
                                       [&](long i, long step, long nw, uint64_t (&w)[2]) { return map_words2(r.mbits0, par, i, step, nw, w); });
        },
        [&]() {
            const ListedArgs<T> r = launch_arguments<ListedArgs<T>>();
            return unclaimed_block<NT>(r.job, busy(r.cand_count), (unsigned)r.ctl[CTL_FRAME] + 1u, bid, reinterpret_cast<int*>(s_word));
        },
        [&](int b) {
            const ListedArgs<T> r = launch_arguments<ListedArgs<T>>();
            const int frame = r.ctl[CTL_FRAME];
            if (take_block(r.job, r.ctl, b, (unsigned)frame + 1u, s_word))
                detect_listed_taken<T, PLC, NT>(r.x, r.S, r.S2, r.mbits0, r.ctl, r.cand, *r.cand_count, r.C, r.Cpx, r.P, r.W, r.tau, r.flags, r.pool_w, r.cand_W, b, blocks, frame & 1);
        },
        [&]() {
            const ListedArgs<T> r = launch_arguments<ListedArgs<T>>();
            extract_own_block<NT>(r.job, r.ctl, bid, reinterpret_cast<const uint64_t*>(lds), epoch, reinterpret_cast<unsigned*>(lds + MAP_STAGE * 8), true);
        });
}

template <typename T>
hipError_t launch_listed_t(const Geom& g, const T* x, T* S, T* S2, uint64_t* mbits, int* ctl, float tau, int flags,
                           const int32_t* cand, const int* cand_count, int cand_cap, int pool_w, int cand_W,
                           DetectJob* job, hipStream_t st, Tm tm)
{
    // channel groups so that a lane holds its (at most 8) channels in registers; few candidates per
    // workgroup, so that a few hundred candidates already spread over the chip
    auto run = [&](auto cs, auto plc) {
        constexpr int CS = decltype(cs)::value, PLC = decltype(plc)::value;
        const unsigned grid = (unsigned)std::min(LISTED_BLOCKS, (cand_cap + PLC - 1) / PLC);
        const bool sh = S2 != nullptr && g.C >= 16 && (g.C & (g.C - 1)) == 0;
        if (job && (job->per = extract_words(job->g, CS * PLC)) > 0) job->nblk = (job->g.Ho * job->g.WWo - 1) / (CS * PLC / 64 * job->per) + 1;
        if (job) job->inv_wwo = map_row_inv((unsigned)job->g.WWo);
        if (job && job->ahead) job->ahead = job->nblk;
        if (job) job->nclaims = (int)grid;
#define CB_LISTED(SH)                                                                                                            \
    if (job && job->nblk)                                                                                                        \
        CB_LAUNCH((detect_listed_extract_kernel<T, CS, PLC, SH>), dim3(grid + (unsigned)job->nblk), dim3(CS * PLC), st, tm,      \
                  (ListedArgs<T>{x, S, S2, mbits, ctl, cand, cand_count, cand_cap, g.C, g.Cs, g.P, g.W, tau, flags, pool_w, cand_W, 0, *job}));  \
    else                                                                                                                         \
        CB_LAUNCH((detect_listed_kernel<T, CS, PLC, SH>), dim3(grid), dim3(CS * PLC), st, tm, x, S, S2, mbits, ctl, cand, cand_count, \
                  cand_cap, g.C, g.Cs, g.P, g.W, tau, flags, pool_w, cand_W)
        if (sh) { CB_LISTED(true); }
        else { CB_LISTED(false); }
#undef CB_LISTED
    };
    typedef std::integral_constant<int, 16> I16;
    if (g.C <= 32)       run(std::integral_constant<int, 4>(), std::integral_constant<int, 64>());
    else if (g.C <= 64)  run(std::integral_constant<int, 8>(), std::integral_constant<int, 32>());
    else if (g.C <= 128) run(I16(), I16());
    else if (g.C <= 256) run(std::integral_constant<int, 32>(), I16());
    else                 run(std::integral_constant<int, 64>(), I16());
    return hipGetLastError();
}

// DET_STREAM_STATE for bfloat16, whose detection stores state and shadow itself: the counts of listed pixels of the frame before,
// from .x to below .y, behind which the state is read past the last-level cache (256 MB).  Behind a frame that wrote most of
// that cache (output, state, shadow; a pixel changed for every 1.25 listed), a state read past it gains nothing and the
// stores of this frame are the slower ones; a state that is not much larger than the cache is better kept in
// it unless a large output pushes it out.  Frames, us, past the cache / through it: 128 -> 128, 3x3, 1080p (531 MB) 170 / 182 at 0.1 %
// of the pixels changed, 220 / 242 at 1, 341 / 377 at 6, 450 / 454 at 10, 641 / 598 at 20, 977 / 909 at 50; at 900x1600 (368 MB) 128 / 136
// at 0.2 %, 298 / 332 at 10, 384 / 387 at 15, 543 / 506 at 30; 64 -> 128 at 1080p (265 MB) 97 / 89 at 0.2 %, 120 / 116 at 1, 154 / 157 at 3,
// 251 / 302 at 10, 367 / 360 at 15, 504 / 475 at 30; 32 -> 64 at 1440x2560 (236 MB) 106 / 90 at 1 %, 140 / 130 at 3, 177 / 184 at 6, 214 / 256
// at 10, 436 / 411 at 30; 64 -> 96 at 1080p 173 / 189 at 5; 128 -> 64 at 720x1280 (236 MB) 106 / 86 at 1 %, 172 / 156 at 10, 200 / 186 at 15; 64 -> 64 at 900x1280 (147 MB) 69 / 61 at 1 %,
// 120 / 100 at 10, 195 / 176 at 30.
int2 state_read_once(const Geom& g, int esz, bool shadow)
{
    const double state = (double)g.C * g.P * esz, out_px = (double)g.O * esz;
    const double from = state >= 300e6 ? 0.0 : state >= 200e6 ? 23e6 / out_px : 2e9;
    const double below = 160e6 / (out_px + 0.8 * g.C * esz * (shadow ? 2 : 1));
    return make_int2((int)std::min(from, 2e9), (int)std::min(below, 2e9));
}

template <typename T>
hipError_t launch_t(const Geom& g, const T* x, T* S, T* S2, uint64_t* mbits, int* ctl, float tau, int flags,
                    DetectJob* job, hipStream_t st, Tm tm)
{
    const int P = g.P;
    const int2 stream = state_read_once(g, sizeof(T), S2 != nullptr);
    const size_t valign = 4 * sizeof(T);
    // few pixels: one pixel per lane keeps more wavefronts busy than four
    // (with a shadow to update, more than 128 channels take the one-pixel-per-lane variants, which
    // stage the shadow rows through LDS; the looped variant writes them element by element)
    // 33 - 64 float32 channels: one pixel per lane on large maps too.  Workgroups of a quarter of the pixels
    // at 30 instead of 72 registers (four resident per compute unit instead of three) drain sooner at
    // the end of the launch, and the kernels behind it start sooner: 64 channels at 480x640, frame
    // 44.9 -> 42.4 - 42.7 us (two pixels per lane: 43.1 - 43.4 us); the kernel itself 26.9 -> 24.1 - 25.2 us.  No gain
    // for 128 channels (1080p) or for the first layers' 3 channels, so only here.
    const bool one_px = sizeof(T) == 4 && g.C > 32 && g.C <= 64;
    // Four pixels per lane otherwise, from 65 536 pixels on.  bfloat16, whose single pixels are 2-byte loads, from 32 768 on
    // and whatever the alignment (64 channels at 271x435 13.8 -> 7.5 us, 128 channels at 1053x1822 398 -> 184 us).  One against
    // four pixels per lane on either side of that line, odd planes: 128 channels 8.0 against 9.5 us at 171x171, 12.0 against 8.5 at
    // 181x182, 12.7 against 8.7 at 200x201; 64 channels 6.3 / 6.7, 6.5 / 6.0, 6.7 / 6.1; up to 16 channels no difference.  float32 gains nothing from unaligned loads
    // (32 channels at 557x803: 25.1 us either way), and the looped variant for more than 128 channels wants aligned ones.
    const bool aligned = P % 4 == 0 && (uintptr_t)x % valign == 0 && (uintptr_t)S % valign == 0;
    const int regs4 = sizeof(T) == 2 ? 256 : 128;         // channels that the variants with four pixels per lane hold in registers
    const bool vec4 = P >= (sizeof(T) == 4 ? 65536 : 32768) && !one_px &&
                      (aligned || (sizeof(T) == 2 && g.C <= regs4)) && (g.C <= regs4 || (P >= 65536 && !(S2 != nullptr && g.C <= 512)));
    if (vec4) launch_v<T, 4>(x, S, S2, mbits, ctl, g.C, g.Cs, P, tau, flags, stream, job, st, tm);
    else      launch_v<T, 1>(x, S, S2, mbits, ctl, g.C, g.Cs, P, tau, flags, stream, job, st, tm);
    return hipGetLastError();
}

}  // namespace

static hipError_t launch_any(const Geom& g, const void* x, void* S, void* S2, uint64_t* mbits, int* ctl, float tau, int flags, DetectJob* job,
                             hipStream_t st, Tm tm)
{
    // the pixels of a shadow are whole 16-byte pieces
    if (S2 && (g.Cs < g.C || g.Cs % (g.bf16 ? 8 : 4) != 0)) return hipErrorInvalidValue;
    if (g.bf16)
        return launch_t<uint16_t>(g, (const uint16_t*)x, (uint16_t*)S, (uint16_t*)S2, mbits, ctl, tau, flags, job, st, tm);
    return launch_t<float>(g, (const float*)x, (float*)S, (float*)S2, mbits, ctl, tau, flags, job, st, tm);
}

hipError_t launch_detect(const Geom& g, const void* x, void* S, void* S2, uint64_t* mbits, int* ctl,
                         float tau, int flags, hipStream_t st, Tm tm)
{
    return launch_any(g, x, S, S2, mbits, ctl, tau, flags, nullptr, st, tm);
}

size_t detect_mail_bytes(const Geom& g) { return ((size_t)g.P + 63) / 64 * (g.P < 8192 ? 32 : 16); }

// a word for each of: 64 pixels (a workgroup of one pixel a lane, or a wavefront of one that has one channel group), 16 of small maps, 2 048 workgroups of
// detection at listed pixels
size_t detect_claim_bytes(const Geom& g) { return 4 * (size_t)claim_words(std::max(((unsigned)g.P + 63u) / 64u, (unsigned)LISTED_BLOCKS)); }

// (at least 64 words a workgroup)
size_t detect_look_bytes(const Geom& g) { return ((size_t)g.Ho * g.WWo / 64 + 1) * 8; }

hipError_t launch_detect_extract(const Geom& g, const void* x, void* S, void* S2, uint64_t* mbits, int* ctl, float tau, int flags,
                                 DetectJob job, hipStream_t st, Tm tm, bool* extracted)
{
    job.nblk = 0;
    const hipError_t e = launch_any(g, x, S, S2, mbits, ctl, tau, flags, &job, st, tm);
    *extracted = job.nblk > 0;
    return e;
}

hipError_t launch_state_apply(const Geom& g, const void* x, void* S, void* S2, const uint64_t* mbits, const int* ctl,
                              hipStream_t st, Tm tm)
{
    const int nwords = (g.P + 63) / 64;
    const unsigned grid = (unsigned)std::min(nwords, 8192);
    if (g.bf16)
        CB_LAUNCH(state_apply_kernel<uint16_t>, dim3(grid), dim3(256), st, tm, (const uint16_t*)x, (uint16_t*)S, (uint16_t*)S2,
                  mbits, ctl, g.C, g.Cs, g.P, nwords);
    else
        CB_LAUNCH(state_apply_kernel<float>, dim3(grid), dim3(256), st, tm, (const float*)x, (float*)S, (float*)S2, mbits, ctl,
                  g.C, g.Cs, g.P, nwords);
    return hipGetLastError();
}

hipError_t launch_shadow_rebuild(const Geom& g, const void* S, void* S2, hipStream_t st)
{
    const long tiles = (((long)g.P + 63) / 64) * ((g.C + 63) / 64);
    const unsigned grid = (unsigned)std::min(tiles, 8192L);
    if (g.bf16)
        hipLaunchKernelGGL(shadow_rebuild_kernel<uint16_t>, dim3(grid), dim3(256), 0, st, (const uint16_t*)S, (uint16_t*)S2,
                           g.C, g.Cs, g.P);
    else
        hipLaunchKernelGGL(shadow_rebuild_kernel<float>, dim3(grid), dim3(256), 0, st, (const float*)S, (float*)S2, g.C, g.Cs, g.P);
    return hipGetLastError();
}

static hipError_t launch_listed(const Geom& g, const void* x, void* S, void* S2, uint64_t* mbits, int* ctl, float tau, int flags,
                                const int32_t* cand, const int* cand_count, int cand_cap, int pool_w, int cand_W, DetectJob* job, hipStream_t st, Tm tm)
{
    if (cand_cap < 1) return hipErrorInvalidValue;
    if (g.bf16)
        return launch_listed_t<uint16_t>(g, (const uint16_t*)x, (uint16_t*)S, (uint16_t*)S2, mbits, ctl, tau,
                                         flags, cand, cand_count, cand_cap, pool_w, cand_W, job, st, tm);
    return launch_listed_t<float>(g, (const float*)x, (float*)S, (float*)S2, mbits, ctl, tau, flags, cand,
                                  cand_count, cand_cap, pool_w, cand_W, job, st, tm);
}

hipError_t launch_detect_listed(const Geom& g, const void* x, void* S, void* S2, uint64_t* mbits, int* ctl,
                                float tau, int flags, const int32_t* cand, const int* cand_count, int cand_cap,
                                int pool_w, int cand_W, hipStream_t st, Tm tm)
{
    return launch_listed(g, x, S, S2, mbits, ctl, tau, flags, cand, cand_count, cand_cap, pool_w, cand_W, nullptr, st, tm);
}

hipError_t launch_detect_listed_extract(const Geom& g, const void* x, void* S, void* S2, uint64_t* mbits, int* ctl,
                                        float tau, int flags, const int32_t* cand, const int* cand_count, int cand_cap,
                                        int pool_w, int cand_W, DetectJob job, hipStream_t st, Tm tm, bool* extracted)
{
    job.nblk = 0;
    const hipError_t e = launch_listed(g, x, S, S2, mbits, ctl, tau, flags, cand, cand_count, cand_cap, pool_w, cand_W, &job, st, tm);
    *extracted = job.nblk > 0;
    return e;
}

}  // namespace cb
