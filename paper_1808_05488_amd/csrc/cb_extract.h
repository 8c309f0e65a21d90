// Device functions of the dilation (Sec. III-A Eq. 4) and of the index extraction ("Change Indexes Extraction") that more than one
// kernel runs: the kernels of cb_compact.hip, and the fused kernel, whose first workgroups can extract the next layer's list.
#pragma once
#include "cb_claim.h"
#include "cb_kernels.h"

namespace cb {

namespace {

// 64-bit word wi of a bit map.  OWN: `w` holds the two input maps of a layer that detects its own
// changes, interleaved word by word (word wi of the map of frame parity p at index 2*wi + p).  One
// 16-byte load brings word wi of both; sel (the frame parity, which may still be on its way from
// memory when the load is issued) picks.  Otherwise `w` is one plain map.
template <bool OWN>
__device__ __forceinline__ uint64_t map_word(const uint64_t* __restrict__ w, long wi, int sel)
{
    if (OWN) {
        const ulonglong2 p = reinterpret_cast<const ulonglong2*>(w)[wi];
        return (sel & 1) ? p.y : p.x;
    }
    return w[wi];
}

template <bool OWN>
__device__ __forceinline__ bool test_bit(const uint64_t* __restrict__ bits, long bit, int sel)
{
    return (map_word<OWN>(bits, bit >> 6, sel) >> (bit & 63)) & 1ull;
}

// Where the words of the input map come from: memory ...
template <bool OWN>
struct MapInMemory {
    const uint64_t* w;
    int sel;
    __device__ __forceinline__ uint64_t operator()(long wi) const { return map_word<OWN>(w, wi, sel); }
};
// ... or the part of it that a workgroup has staged in LDS (words first, first + 1, ...).
struct MapInLds {
    const uint64_t* w;
    long first;
    __device__ __forceinline__ uint64_t operator()(long wi) const { return w[wi - first]; }
};

// Bits q .. q + 127 (q < 64) of three consecutive words, with 32-bit shifts over two registers: four and five selections, where 64-bit shifts
// take four, of several cycles each, and as many selections for q = 0.  (A 64-bit shift by an amount in the last register of a kernel's
// allocation, v39 of 40, took that amount from register 0 now and then: gfx90a's compiler avoids the form, gfx950's does not.
// tests/test_shift_amounts.py looks for it in every kernel.)
__device__ __forceinline__ void window(const uint64_t (&v)[3], unsigned q, uint64_t& lo, uint64_t& hi)
{
    uint32_t w[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        const uint32_t a = (uint32_t)(v[i >> 1] >> (32 * (i & 1))), b = (uint32_t)(v[(i + 1) >> 1] >> (32 * ((i + 1) & 1)));
        w[i] = q & 32u ? b : a;
    }
    uint32_t r[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = __builtin_amdgcn_alignbit(w[i + 1], w[i], q & 31u);
    lo = (uint64_t)r[1] << 32 | r[0];
    hi = (uint64_t)r[3] << 32 | r[2];
}

// Bit q (q = 0..63) = OR over the filter footprint of an output whose receptive field's top-left
// pixel is (y0, x0 + q); pixels outside the image read as zero.  -63 <= x0.  The filter's rows are
// OR-ed first, as 128-column windows (their column limits are the same for every row), the columns
// afterwards, once, by doubling: kw shifts become log2(kw).  The map has at least two words of
// slack behind its last used word; the window is at most 64 + 30 columns wide.
// KB: filter rows per batch of reads.
template <int KB, typename WORDS>
__device__ __forceinline__ uint64_t fires_rows(const Geom& g, const WORDS& words, long pitch, int y0, int x0)
{
    int a = x0 > 0 ? x0 : 0;
    const int pre = a - x0;
    const int len = (x0 + 128 < g.W ? x0 + 128 : g.W) - a;
    if (a > g.W - 1) a = g.W - 1;                      // keep the address inside the row; len <= 0 masks it
    uint64_t lo = 0, hi = 0;
    // filter rows in batches: their reads are issued before the first use
    for (int j0 = 0; j0 < g.kh; j0 += KB) {
        uint64_t v[KB][3];
        int sh[KB];
#pragma unroll
        for (int u = 0; u < KB; ++u) {
            const int yi = y0 + j0 + u;
            const bool valid = j0 + u < g.kh && yi >= 0 && yi < g.H;
            const int yr = j0 + u < g.kh ? yi : y0 + j0;   // (a row beyond the filter's last repeats the batch's first)
            const int yc = yr < 0 ? 0 : (yr >= g.H ? g.H - 1 : yr);
            const long bit = (long)yc * pitch + a;
            sh[u] = valid ? (int)(bit & 63) : -1;
#pragma unroll
            for (int k = 0; k < 3; ++k) v[u][k] = words((bit >> 6) + k);
        }
#pragma unroll
        for (int u = 0; u < KB; ++u) {
            uint64_t l, h;
            window(v[u], (unsigned)sh[u] & 63u, l, h);
            lo |= sh[u] >= 0 ? l : 0ull;
            hi |= sh[u] >= 0 ? h : 0ull;
        }
    }
    lo &= len >= 64 ? ~0ull : (len > 0 ? (1ull << len) - 1ull : 0ull);
    hi &= len >= 128 ? ~0ull : (len > 64 ? (1ull << (len - 64)) - 1ull : 0ull);
    if (pre) { hi = (hi << pre) | (lo >> (64 - pre)); lo <<= pre; }
    int n = 1;                                         // bit q holds columns q .. q + n - 1
    while (2 * n <= g.kw) { lo |= (lo >> n) | (hi << (64 - n)); hi |= hi >> n; n *= 2; }
    if (n < g.kw) { const int r = g.kw - n; lo |= (lo >> r) | (hi << (64 - r)); }
    return lo;
}

// The same from the part of a map that is staged in LDS (its first bit: first_bit), for whole wavefronts: 2^share groups of 64 >> share lanes hold the same outputs,
// each takes every 2^share-th filter row from `group` on, and all have the result.  32-bit windows over single words of the map; a window is at most
// 64 + 30 columns.  (fires_rows there: 1.0 us with 3 rows, 1.6 with 9, of which most is the arithmetic of a lone wavefront.)
__device__ __forceinline__ uint64_t fires_shared(const Geom& g, const uint64_t* lds, unsigned first_bit, int y0, int x0, int share, int group)
{
    const uint32_t* const map = reinterpret_cast<const uint32_t*>(lds);
    int a = x0 > 0 ? x0 : 0;
    const int pre = a - x0, len = g.W - a;
    if (a > g.W - 1) a = g.W - 1;                      // keep the address inside the row; len <= 0 masks it
    uint32_t r0 = 0, r1 = 0, r2 = 0;
    for (int j0 = 0; j0 < g.kh; j0 += 2 << share) {
        uint32_t v[2][4];
        unsigned sh[2];
        bool in[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int j = j0 + group + (u << share), yi = y0 + j;
            in[u] = j < g.kh && yi >= 0 && yi < g.H;
            const int yr = y0 + (j < g.kh ? j : g.kh - 1), yc = yr < 0 ? 0 : (yr >= g.H ? g.H - 1 : yr);
            const unsigned bit = (unsigned)yc * (unsigned)g.W + (unsigned)a - first_bit;
            sh[u] = bit & 31u;
#pragma unroll
            for (int k = 0; k < 4; ++k) v[u][k] = map[(bit >> 5) + k];
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint32_t on = in[u] ? ~0u : 0u;
            r0 |= __builtin_amdgcn_alignbit(v[u][1], v[u][0], sh[u]) & on;
            r1 |= __builtin_amdgcn_alignbit(v[u][2], v[u][1], sh[u]) & on;
            r2 |= __builtin_amdgcn_alignbit(v[u][3], v[u][2], sh[u]) & on;
        }
    }
    auto both = [](auto p) { return p[0] | p[1]; };
    if (share >= 1) {
        r0 = both(__builtin_amdgcn_permlane32_swap(r0, r0, false, false));
        r1 = both(__builtin_amdgcn_permlane32_swap(r1, r1, false, false));
        r2 = both(__builtin_amdgcn_permlane32_swap(r2, r2, false, false));
    }
    if (share >= 2) {
        r0 = both(__builtin_amdgcn_permlane16_swap(r0, r0, false, false));
        r1 = both(__builtin_amdgcn_permlane16_swap(r1, r1, false, false));
        r2 = both(__builtin_amdgcn_permlane16_swap(r2, r2, false, false));
    }
    auto first_bits = [](int n) { return n >= 32 ? ~0u : n > 0 ? (1u << n) - 1u : 0u; };
    r0 &= first_bits(len);
    r1 &= first_bits(len - 32);
    r2 &= first_bits(len - 64);
    if (pre) {                                         // at most pad <= 31 columns
        r2 = __builtin_amdgcn_alignbit(r2, r1, 32 - pre);
        r1 = __builtin_amdgcn_alignbit(r1, r0, 32 - pre);
        r0 <<= pre;
    }
    auto or_shifted = [&](int n) {
        r0 |= __builtin_amdgcn_alignbit(r1, r0, n);
        r1 |= __builtin_amdgcn_alignbit(r2, r1, n);
        r2 |= r2 >> n;
    };
    int n = 1;                                         // bit q holds columns q .. q + n - 1
    while (2 * n <= g.kw) { or_shifted(n); n *= 2; }
    if (n < g.kw) or_shifted(g.kw - n);
    return (uint64_t)r1 << 32 | r0;
}

template <typename WORDS>
__device__ __forceinline__ uint64_t fires64(const Geom& g, const WORDS& words, long pitch, int y0, int x0)
{
    return g.kh == 1 ? fires_rows<1>(g, words, pitch, y0, x0) : fires_rows<4>(g, words, pitch, y0, x0);
}

// bits 0, 2, 4, ... of v squeezed into the lower half
__device__ __forceinline__ uint64_t even_bits(uint64_t v)
{
    v &= 0x5555555555555555ull;
    v = (v | (v >> 1)) & 0x3333333333333333ull;
    v = (v | (v >> 2)) & 0x0F0F0F0F0F0F0F0Full;
    v = (v | (v >> 4)) & 0x00FF00FF00FF00FFull;
    v = (v | (v >> 8)) & 0x0000FFFF0000FFFFull;
    return (v | (v >> 16)) & 0x00000000FFFFFFFFull;
}

// One word of the dilated map: output row yo, columns 64*wo .. 64*wo+63.  A strided layer takes every
// s-th bit of the words a layer of stride 1 would have there: s window words per output word, all of
// them words from the map.  (Testing the map bit by bit, kh*kw dependent loads per output, took 248 us
// of a 273 us frame for 48 -> 96 channels, 5x5, stride 2 at 241x323.)  Beyond a stride of 64 the
// outputs lie in different words anyway, one window each.
template <typename WORDS>
__device__ __forceinline__ uint64_t dilated_word_t(const Geom& g, const WORDS& words, long pitch, int yo, int wo)
{
    const int nvalid = g.Wo - 64 * wo < 64 ? g.Wo - 64 * wo : 64;
    const uint64_t vmask = nvalid == 64 ? ~0ull : ((1ull << nvalid) - 1ull);
    const int y0 = yo * g.s - g.p;
    if (g.s == 1) return fires64(g, words, pitch, y0, 64 * wo - g.p) & vmask;
    uint64_t word = 0;
    if (g.s == 2) {
        const int x0 = 128 * wo - g.p;
        word = even_bits(fires64(g, words, pitch, y0, x0));
        if (nvalid > 32) word |= even_bits(fires64(g, words, pitch, y0, x0 + 64)) << 32;
    } else if (g.s <= 64) {
        // output b is anchored at column b*s of the window; the anchors come in ascending order
        int b = 0;
        for (int t = 0; t < g.s && b < nvalid; ++t) {
            const uint64_t f = fires64(g, words, pitch, y0, 64 * wo * g.s - g.p + 64 * t);
            for (; b < nvalid && b * g.s < 64 * (t + 1); ++b) word |= ((f >> (b * g.s - 64 * t)) & 1ull) << b;
        }
    } else {
        for (int b = 0; b < nvalid; ++b)
            word |= (fires64(g, words, pitch, y0, (64 * wo + b) * g.s - g.p) & 1ull) << b;
    }
    return word & vmask;
}

// own_map: in_bits holds the layer's two interleaved input maps and sel is the frame parity
__device__ __forceinline__ uint64_t dilated_word(const Geom& g, const uint64_t* __restrict__ in_bits, long pitch,
                                                 int yo, int wo, int own_map, int sel)
{
    return own_map ? dilated_word_t(g, MapInMemory<true>{in_bits, sel}, pitch, yo, wo)
                   : dilated_word_t(g, MapInMemory<false>{in_bits, 0}, pitch, yo, wo);
}

// Input words under words it0 .. it0 + NT - 1 (below items) of the dilated map: n from `first` on.
template <int NT> __device__ __forceinline__ void block_range(const Geom& g, long pitch, int it0, int items, long& first, long& n)
{
    const int ilast = (it0 + NT < items ? it0 + NT : items) - 1;
    const int y0 = it0 / g.WWo, y1 = ilast / g.WWo;
    int r0 = y0 * g.s - g.p, r1 = y1 * g.s - g.p + g.kh - 1;
    // (rows outside the image are read at its first / last row)
    r0 = r0 < 0 ? 0 : (r0 > g.H - 1 ? g.H - 1 : r0);
    r1 = r1 < 0 ? 0 : (r1 > g.H - 1 ? g.H - 1 : r1);
    first = ((long)r0 * pitch) >> 6;
    n = ((((long)r1 * pitch + g.W - 1) >> 6) + 3) - first;                // a window reads two words past its first
}

// Words it0 .. it0 + NT - 1 of the dilated map, one per thread of a workgroup of NT threads (0 beyond the
// last).  The rows of the input map under them are one contiguous range of words: the workgroup stages it in
// LDS with one round of loads, and the windows, which overlap kh times, are cut out there (7x7 at 240x320:
// 8.4 -> 7.6 us for dilation and list, 9x9 10.7 -> 7.2).  Filters of up to four rows at stride 1 issue all their
// loads in one batch anyway and go without the detour (1x1: 5.0 us, staged 5.8); ranges of
// more than CAP words (large strides, very wide filters on narrow maps) are read from memory too.
// Called by all threads of the workgroup.
template <int NT, int CAP>
__device__ __forceinline__ uint64_t dilated_block_word(const Geom& g, const uint64_t* __restrict__ in_bits, long pitch,
                                                       int it0, int items, int own_map, int sel, uint64_t* s_map)
{
    const int tid = threadIdx.x, it = it0 + tid;
    long first, n;
    block_range<NT>(g, pitch, it0, items, first, n);
    const int yo = it / g.WWo, wo = it - yo * g.WWo;
    if ((g.s == 1 && g.kh <= 4) || n > CAP) return it < items ? dilated_word(g, in_bits, pitch, yo, wo, own_map, sel) : 0ull;
    if (own_map) {
        for (int i = tid; i < (int)n; i += NT) s_map[i] = map_word<true>(in_bits, first + i, sel);
    } else {
        for (int i = tid; i < (int)n; i += NT) s_map[i] = map_word<false>(in_bits, first + i, 0);
    }
    __syncthreads();
    return it < items ? dilated_word_t(g, MapInLds{s_map, first}, pitch, yo, wo) : 0ull;
}

// Inclusive prefix sum over the 64 lanes of a wavefront with data-parallel-primitive moves: shifts by
// 1, 2, 4, 8 inside each row of 16 lanes, then lane 15 of a row broadcast into the next row and lane 31
// into the upper half (lanes without a source add 0).  Six register-to-register steps; the same scan
// through general shuffles costs six LDS round trips.
__device__ __forceinline__ int wave_inclusive_scan(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
    return v;
}
// ... and the sum over the wavefront, in every lane: the last lane of that scan
__device__ __forceinline__ int wave_sum(int v) { return __builtin_amdgcn_readlane(wave_inclusive_scan(v), 63); }

// OR over the wavefront, in every lane
__device__ __forceinline__ int wave_or(int v)
{
    v |= __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
    v |= __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v |= __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v |= __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v |= __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
    v |= __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    return __builtin_amdgcn_readlane(v, 63);
}

// Index-list entries of the 64 words held by a wavefront (word, its exclusive offset, the
// pixel index of its bit 0).  PER_LANE = false: the whole wavefront expands one non-empty word
// at a time (coalesced stores, a handful of cross-lane reads per word) -- the faster form
// when the words are spread over many compute units.  PER_LANE = true: every lane walks the
// bits of its own word, no cross-lane traffic -- the faster form in the one-workgroup kernel,
// where sixteen wavefronts share one compute unit's cross-lane hardware.
template <bool PER_LANE>
__device__ __forceinline__ void expand_words(uint64_t word, int off, int pixbase, int32_t* __restrict__ idx, int lane)
{
    if (PER_LANE) {
        while (word) {
            idx[off++] = pixbase + __builtin_ctzll(word);
            word &= word - 1;
        }
        return;
    }
    uint64_t nz = __ballot(word != 0);
    while (nz) {
        // (nz comes from a ballot, so src is the same in every lane: plain lane reads into scalar registers,
        // not the cross-lane permutes of a general shuffle, which cost an LDS round trip each; the word is the mask of the
        // lanes that store, and what precedes a lane's bit two instructions)
        const int src = __ffsll((long long)nz) - 1;
        nz &= nz - 1;
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)word, src);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(word >> 32), src);
        const int o = __builtin_amdgcn_readlane(off, src);
        const int pb = __builtin_amdgcn_readlane(pixbase, src);
        const int at = (int)__builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, (unsigned)o));
        if (__builtin_amdgcn_inverse_ballot_w64(((uint64_t)hi << 32) | lo)) idx[at] = pb + lane;
    }
}

// A layer that detects its own changes keeps two input maps (interleaved word by word, see
// map_word) and two changed-pixel counters, used by alternate frames: change detection fills the
// pair that the frame count on the device (CTL_FRAME, advanced by the index extraction once per
// frame) selects, and the index extraction clears the other pair for the next frame.  Nothing about
// this lives on the host, so captured launches replay correctly whatever the number of frames in a
// capture.  A layer that takes its map from its producer (own_map == 0) has one plain map and
// nothing to clear.
__device__ __forceinline__ int frame_parity(const int* ctl, int own_map) { return own_map ? (ctl[CTL_FRAME] & 1) : 0; }
// the other map and the other counter start the next frame empty
__device__ __forceinline__ void clear_other_map(uint64_t* maps, int* ctl, int par, int clear_words, int first, int step)
{
    if (first < NIN_SLOTS) *nin_counter(ctl, (unsigned)first, par ^ 1) = 0;
    for (int i = first; i < clear_words; i += step) maps[2 * i + (par ^ 1)] = 0;
}

// word `it` of the dilated map of a full update: every output
__device__ __forceinline__ uint64_t full_word(const Geom& g, int it)
{
    const int nvalid = g.Wo - 64 * (it % g.WWo);
    return nvalid >= 64 ? ~0ull : ((1ull << nvalid) - 1ull);
}

// Words of the input map a workgroup can stage: 256 output words of a 1080p layer with stride 1 and a 31-row
// filter need 1 200 words, of a VGA layer with stride 2 and 7 rows 1 092 (16 KB).  The one-workgroup kernel, up to 1024
// output words, stages maps of up to 4 605 words whole (36 KB); that of a VGA layer with stride 3 or 4, 4 802 words, is
// read from memory.
constexpr int MAP_STAGE = 2048, MAP_STAGE_SMALL = 4608;

// The end of a frame's extraction, by one thread, when nobody of the launch reads the epoch, the frame count or the arrivals any more.
__device__ __forceinline__ void finish_frame(int* ctl, unsigned epoch, int own_map, bool arrivals)
{
    ctl[CTL_DONE] = 0;
    ctl[CTL_BEGUN] = 0;
    ctl[CTL_EPOCH] = (int)epoch;
    if (arrivals)
#pragma unroll 1
        for (int q = 0; q < ARRIVE_SLOTS; ++q) ctl[CTL_ARRIVE + q * NIN_STRIDE] = 0;
    if (own_map) ctl[CTL_FRAME] = ctl[CTL_FRAME] + 1;
}
// epoch of the launch that follows the one of epoch `last` (0 is what never-written slots hold)
__device__ __forceinline__ unsigned next_epoch(unsigned last) { return last + 1u ? last + 1u : 1u; }

// atomics of cb_claim.h, past the caches of an XCD
struct DeviceMem {
    __device__ __forceinline__ unsigned exchange(unsigned* p, unsigned v) const { return __hip_atomic_exchange(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ __forceinline__ int add(int* p, int v) const
    {
        int old = __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("" : "+v"(old) :: "memory");            // it has returned
        return old;
    }
};

// ... whose answer is waited for where it is used
struct DeviceMemLater {
    __device__ __forceinline__ int add(int* p, int v) const { return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
};

// The second half of the single-pass extraction, for workgroup bid of nblk: scan over the workgroups' words and index write.
// word: this thread's word of the dilated map, pixbase the pixel of its bit 0; epoch_ld (thread 0): CTL_EPOCH as it was at launch;
// recount(b): the set bits in workgroup b's 256 words, from the input map alone; small: LDS, ONE_PASS_SMALL words.
// NW: wavefronts of a workgroup.  LIMITED: the wait for another workgroup's count ends after spin_limit polls and the count is
// recomputed; otherwise workgroups of lower numbers have begun (extraction_number in cb_claim.h), and the wait ends with the count.
template <int NW> __host__ __device__ constexpr int one_pass_small() { return 2 * NW + 1; }
constexpr int ONE_PASS_SMALL = one_pass_small<4>();
template <int NW = 4, bool LIMITED = true, typename RECOUNT>
__device__ __forceinline__ void one_pass_tail(uint64_t word, int pixbase, unsigned epoch_ld, int32_t* __restrict__ idx, int* __restrict__ ctl,
                                              unsigned long long* __restrict__ look, int own_map, int bid, int nblk, int spin_limit,
                                              unsigned* small, RECOUNT&& recount, bool arrivals = false)
{
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    int* const wtot = reinterpret_cast<int*>(small);
    int* const red = wtot + NW;
    unsigned& s_epoch = small[2 * NW];
    const int cnt = __popcll(word);
    const int inc = wave_inclusive_scan(cnt);                  // inclusive scan inside the wavefront
    if (lane == 63) wtot[wv] = inc;
    if (tid == 0) s_epoch = next_epoch(epoch_ld);
    __syncthreads();
    const unsigned epoch = s_epoch;
    if (tid == 0) {
        unsigned total = 0;
#pragma unroll
        for (int q = 0; q < NW; ++q) total += (unsigned)wtot[q];
        __hip_atomic_store(&look[bid], ((unsigned long long)epoch << 32) | total, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    // counts of all earlier workgroups (count and epoch travel in one word: no ordering between words needed)
    int part = 0;
    for (int b = tid; b < bid; b += 64 * NW) {
        unsigned long long v = 0;
        int spins = 0;
        for (;;) {
            v = __hip_atomic_load(&look[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if ((unsigned)(v >> 32) == epoch) break;
            if constexpr (LIMITED)
                if (++spins > spin_limit) {
                    v = (unsigned long long)(unsigned)recount(b);
                    atomicAdd(&ctl[CTL_RECOUNTS], 1);
                    break;
                }
            __builtin_amdgcn_s_sleep(1);
        }
        part += (int)(unsigned)v;
    }
    part = wave_sum(part);
    if (lane == 0) red[wv] = part;
    __syncthreads();
    int off = 0;
#pragma unroll
    for (int q = 0; q < NW; ++q) off += red[q];
    for (int q = 0; q < wv; ++q) off += wtot[q];
    off += inc - cnt;                                        // exclusive offset of this thread's word
    if (bid == nblk - 1 && tid == 64 * NW - 1) ctl[CTL_COUNT] = off + cnt;

    // (what ends the frame reads nothing of the list: the answer, a round trip of 0.8 us, is on its way beside the list's stores)
    int through = 0;
    if (tid == 0) through = DeviceMemLater().add(&ctl[CTL_DONE], 1);
    expand_words<false>(word, off, pixbase, idx, lane);
    if (tid == 0 && extraction_last(through, nblk)) finish_frame(ctl, epoch, own_map, arrivals);
}

// Word wi (row-padded) of the 2 x 2 pooled map of a producer's row-padded dilated map: OR over the windows, border windows clipped.
__device__ __forceinline__ uint64_t pooled_word(const uint64_t* __restrict__ mt, int Ho, int WWo, int yp, int wp)
{
    // OR the two producer rows, OR neighbouring bit pairs, squeeze the even bits together (bits beyond the row's end are 0)
    uint64_t v[2] = {0, 0};
#pragma unroll
    for (int dy = 0; dy < 2; ++dy)
#pragma unroll
        for (int h = 0; h < 2; ++h)
            if (2 * yp + dy < Ho && 2 * wp + h < WWo) v[h] |= mt[(long)(2 * yp + dy) * WWo + 2 * wp + h];
    return even_bits(v[0] | (v[0] >> 1)) | (even_bits(v[1] | (v[1] >> 1)) << 32);
}
// Word wi of the map a consumer takes from its producer: the producer's map, or its pooled form (pooled).
struct MapOfProducer {
    const uint64_t* mt;
    int Ho, WWo, H, WW;
    bool pooled;
    __device__ __forceinline__ uint64_t operator()(long wi) const
    {
        if (!pooled) return mt[wi];
        const int yp = (int)(wi / WW);
        return yp < H ? pooled_word(mt, Ho, WWo, yp, (int)(wi - (long)yp * WW)) : 0ull;
    }
};

// One workgroup (bid of job.nblk, 256 threads) of an extraction; lds: EXTRACT_LDS bytes.
constexpr unsigned EXTRACT_LDS = MAP_STAGE * 8u + ONE_PASS_SMALL * 4u;
__device__ __forceinline__ void extract_block(const ExtractJob& job, int bid, uint64_t* lds)
{
    const Geom& g = job.g;
    const MapOfProducer src{job.in_bits, job.src_Ho, job.src_WWo, g.H, (g.W + 63) / 64, job.pm_bits != nullptr};
    const int tid = threadIdx.x, items = g.Ho * g.WWo, it = bid * 256 + tid;
    const unsigned epoch_ld = tid == 0 ? (unsigned)job.ctl[CTL_EPOCH] : 0u;
    if (src.pooled)
        for (int i = bid * 256 + tid; i < src.H * src.WW; i += job.nblk * 256) job.pm_bits[i] = src(i);
    long first, n;
    block_range<256>(g, job.pitch, bid * 256, items, first, n);
    for (int i = tid; i < (int)n; i += 256) lds[i] = src(first + i);
    __syncthreads();
    const int yo = it / g.WWo, wo = it - yo * g.WWo;
    uint64_t word = 0;
    int pixbase = 0;
    if (it < items) {
        word = dilated_word_t(g, MapInLds{lds, first}, job.pitch, yo, wo);
        job.mt_bits[it] = word;
        pixbase = yo * g.Wo + 64 * wo;
    }
    one_pass_tail<4>(word, pixbase, epoch_ld, job.idx, job.ctl, job.look, 0, bid, job.nblk, job.spin_limit,
                  reinterpret_cast<unsigned*>(lds + MAP_STAGE), [&](int b) {
                      int total = 0;
                      const int hi = b * 256 + 256 < items ? b * 256 + 256 : items;
                      for (int i = b * 256; i < hi; ++i) total += __popcll(dilated_word_t(g, src, job.pitch, i / g.WWo, i % g.WWo));
                      return total;
                  });
}

// The change map of a frame on its way to extracting workgroups of the same launch: units of up to 32 pixels (16 for workgroups of 16
// pixels), each one 64-bit value with the frame's tag above the bits.  A unit travels whole, so its reader needs no other ordering than to see the
// tag, and its writer waits for nothing.  (A count of finished workgroups instead means a wait for two round trips to memory in each
// of them; a fence, needed for plain stores of the map, raised detection from 26 to 344 us on a VGA layer of 64 channels.)
__device__ __forceinline__ void mail_put(uint64_t* mail, long unit, unsigned tag, unsigned bits)
{
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(mail) + unit, ((unsigned long long)tag << 32) | bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// words i and i + step of the map (those from nwords on are 0), from UPW units each; waits for them (limited: for as many polls as are left)
template <int UPW> __device__ __forceinline__ bool mail_words(const uint64_t* mail, long i, long step, long nwords, unsigned tag, uint64_t (&w)[2], bool limited, int& polls)
{
    unsigned long long v[2][UPW];
    for (;;) {
        bool all = true;
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int u = 0; u < UPW; ++u) {
                const long wi = i + k * step < nwords ? i + k * step : i;        // (i itself is below nwords)
                v[k][u] = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(mail) + UPW * wi + u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int u = 0; u < UPW; ++u) all = all && (unsigned)(v[k][u] >> 32) == tag;
        if (all) break;
        if (limited && --polls < 0) return false;
        __builtin_amdgcn_s_sleep(1);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        w[k] = 0;
#pragma unroll
        for (int u = 0; u < UPW; ++u) w[k] |= (uint64_t)(unsigned)v[k][u] << (64 / UPW * u);
        if (i + k * step >= nwords) w[k] = 0;
    }
    return true;
}

// The extraction inside the launch of detection, workgroup bid of job.nblk (NT threads).  A wavefront has job.per words of
// the dilated map, 16 where there are few: dense words are expanded one after the other, and a part of a map that is waited for should be
// small.  Strides 1 and 2 (extract_words in cb_detect.hip).
// First: the part of the input map that its words are made from, into lds (MAP_STAGE words), complete.  fetch2(i, step, nwords, w): words i < nwords and
// i + step of the map, or false if they did not come in time; then so is the result, in all threads.  s_short: a word of LDS of its own.
template <int NT, typename FETCH>
__device__ __forceinline__ bool stage_own_block(const DetectJob& job, int bid, uint64_t* lds, unsigned* s_short, FETCH&& fetch2)
{
    const Geom& g = job.g;
    const int tid = threadIdx.x, items = g.Ho * g.WWo, nwords = (g.P + 63) / 64;
    const int ipb = NT / 64 * job.per, it0 = bid * ipb;                  // words of a workgroup, its first
    // The input rows under this workgroup's words, and those between them and the next workgroup's, so that together the workgroups wait for
    // every word: then all that detect have read the frame count and the last count of listed pixels, which the tail overwrites.
    const int last = (it0 + ipb < items ? it0 + ipb : items) - 1;
    int r0 = (int)map_row((unsigned)it0, job.inv_wwo) * g.s - g.p, r1 = (int)map_row((unsigned)last, job.inv_wwo) * g.s - g.p + g.kh - 1;
    const int next = last + 1 < items ? (int)map_row((unsigned)last + 1u, job.inv_wwo) * g.s - g.p - 1 : g.H - 1;
    r1 = r1 > next ? r1 : next;
    r0 = r0 < 0 ? 0 : (r0 > g.H - 1 ? g.H - 1 : r0);
    r1 = r1 < 0 ? 0 : (r1 > g.H - 1 ? g.H - 1 : r1);
    const long first = ((long)r0 * g.W) >> 6;
    const int n = (int)(((((long)r1 * g.W + g.W - 1) >> 6) + 3) - first);
    if (tid == 0) *s_short = 0;
    __syncthreads();
    bool all = true;
    for (int i = tid; i < n && all; i += 2 * NT) {
        uint64_t w[2] = {0, 0};
        if (first + i < nwords) all = fetch2(first + i, (long)NT, (long)nwords, w);
        lds[i] = w[0];
        if (i + NT < n) lds[i + NT] = w[1];
    }
    if (!all) *s_short = 1;
    __syncthreads();
    return *s_short == 0;
}
// Then: its words, and its part of the list.  epoch_ld (thread 0): CTL_EPOCH; small: one_pass_small 32-bit words of LDS.
template <int NT>
__device__ __forceinline__ void extract_own_block(const DetectJob& job, int* __restrict__ ctl, int bid, const uint64_t* lds, unsigned epoch_ld, unsigned* small, bool arrivals)
{
    const Geom& g = job.g;
    const int tid = threadIdx.x, lane = tid & 63, items = g.Ho * g.WWo;
    const int ipb = NT / 64 * job.per, it0 = bid * ipb;
    // lanes of one word: 64 / per, with a part of the filter's rows each; the first of them holds it
    const int lper = 31 - __builtin_clz((unsigned)job.per), last = (it0 + ipb < items ? it0 + ipb : items) - 1;
    const int it = it0 + (tid >> 6) * job.per + (lane & (job.per - 1)), at = it < last ? it : last;
    const bool mine = lane < job.per && it < items;
    int r0 = (int)map_row((unsigned)it0, job.inv_wwo) * g.s - g.p;       // (as in stage_own_block)
    r0 = r0 < 0 ? 0 : (r0 > g.H - 1 ? g.H - 1 : r0);
    const unsigned first_bit = (unsigned)r0 * (unsigned)g.W & ~63u;
    const int yo = (int)map_row((unsigned)at, job.inv_wwo), wo = at - yo * g.WWo;
    uint64_t word = 0;
    if (job.full) word = full_word(g, at);
    else {
        const int nvalid = g.Wo - 64 * wo < 64 ? g.Wo - 64 * wo : 64;
#pragma unroll 1
        for (int t = 0; t < g.s && 32 * t < g.Wo; ++t) {                 // (the same number for all lanes; the second half of a word beyond the map is masked)
            const uint64_t f = fires_shared(g, lds, first_bit, yo * g.s - g.p, 64 * wo * g.s - g.p + 64 * t, 6 - lper, lane >> lper);
            word |= g.s == 1 ? f : even_bits(f) << (32 * t);
        }
        word &= nvalid == 64 ? ~0ull : ((1ull << nvalid) - 1ull);
    }
    if (!mine) word = 0;
    else job.mt_bits[it] = word;
    const int pixbase = yo * g.Wo + 64 * wo;
    one_pass_tail<NT / 64, false>(word, pixbase, epoch_ld, job.idx, ctl, job.look, 1, bid, job.nblk, 0, small, [](int) {}, arrivals);
}

// Some block among the first n that nobody has claimed in this frame, in all threads of the workgroup, or -1; each workgroup looks from a place of its own on.
// s_found: a word of LDS of its own.
template <int NT> __device__ __forceinline__ int unclaimed_block(const DetectJob& job, int n, unsigned tag, int bid, int* s_found)
{
    const int from = (int)((long)n * bid / job.nblk);
    for (int i = 0; i < n; i += NT) {
        if (threadIdx.x == 0) *s_found = n;
        __syncthreads();
        const int o = i + (int)threadIdx.x, c = from + o < n ? from + o : from + o - n;
        if (o < n && __hip_atomic_load(job.claims + claim_index((unsigned)c, (unsigned)job.nclaims), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != tag) atomicMin(s_found, o);
        __syncthreads();
        const int found = *s_found;
        __syncthreads();
        if (found < n) return __builtin_amdgcn_readfirstlane(from + found < n ? from + found : from + found - n);
    }
    return -1;
}

// The arguments of a kernel whose only parameter is an A, loaded once more where this is called: what only a rare path needs need not be held in registers on
// the way there.
template <typename A> __device__ __forceinline__ A launch_arguments()
{
    typedef const __attribute__((address_space(4))) unsigned* words;
    words p = (words)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    static_assert(sizeof(A) % 4 == 0, "whole words");
    unsigned w[sizeof(A) / 4];
#pragma unroll
    for (unsigned i = 0; i < sizeof(A) / 4; ++i) w[i] = p[i];
    A a;
    __builtin_memcpy(&a, w, sizeof(A));
    return a;
}

// What workgroup number blockIdx.x does: extracts, or detects, as number own of n.
struct Role { bool extracts; int own, n; };
__device__ __forceinline__ Role role_of(const DetectJob& job)
{
    const int n = (int)gridDim.x - job.nblk, own = (int)blockIdx.x - job.ahead;
    return Role{own < 0 || own >= n, own, n};
}
// An extracting workgroup begins: its number.  s_word: a word of LDS of its own.
__device__ __forceinline__ int begin_extraction(int* ctl, int nblk, unsigned* s_word)
{
    if (nblk == 1) return 0;                     // (without the round trip)
    if (threadIdx.x == 0) *s_word = (unsigned)extraction_number(DeviceMem(), &ctl[CTL_BEGUN]);
    __syncthreads();
    const int bid = (int)__builtin_amdgcn_readfirstlane(*s_word);
    __syncthreads();
    return bid;
}

// Claims a block for a workgroup other than its own: whether it has it now, in all threads.  s_word: a word of LDS of its own.
__device__ __forceinline__ bool take_block(const DetectJob& job, int* ctl, int b, unsigned tag, unsigned* s_word)
{
    if (threadIdx.x == 0) {
        const bool lost = claim_block(DeviceMem(), job.claims + claim_index((unsigned)b, (unsigned)job.nclaims), tag, &ctl[CTL_DONE], true) == tag;
        if (lost) claim_lost(DeviceMem(), &ctl[CTL_DONE], job.nblk);         // (never the end of the frame: this workgroup is not through)
        else atomicAdd(&ctl[CTL_RECOUNTS], 1);
        *s_word = lost ? 1u : 0u;
    }
    __syncthreads();
    const bool mine = *s_word == 0;
    __syncthreads();
    return mine;
}

// Detection at listed pixels sets single bits of a cleared map with atomics, which are complete when their old value has come back; a workgroup
// that had pixels then adds itself to one of the counters.  (A few hundred workgroups: one counter would queue them up for 3 us.)
__device__ __forceinline__ void arrive(int* ctl, unsigned b)
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0F70);          // vmcnt(0): every atomic of this wavefront has returned
    asm volatile("" ::: "memory");
    __hip_atomic_fetch_add(ctl + CTL_ARRIVE + (b % ARRIVE_SLOTS) * NIN_STRIDE, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// called by whole workgroups: waits for `expected` workgroups (limited: so many polls, then false); s_short: a word of LDS of its own
__device__ __forceinline__ bool await_arrivals(const int* ctl, int expected, bool limited, int polls, unsigned* s_short)
{
    const int lane = threadIdx.x & 63;
    if (threadIdx.x < 64)
        for (;;) {
            const int n = lane < ARRIVE_SLOTS ? __hip_atomic_load(ctl + CTL_ARRIVE + lane * NIN_STRIDE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
            const bool all = wave_sum(n) >= expected, stop = all || (limited && --polls < 0);
            if (stop && lane == 0) *s_short = all ? 0u : 1u;
            if (stop) break;
            __builtin_amdgcn_s_sleep(1);
        }
    __syncthreads();
    const bool all = *s_short == 0;
    __syncthreads();
    return all;
}
// words i and i + step of the map of parity par (interleaved with the other one), past the caches that do not see other XCDs' atomics
__device__ __forceinline__ bool map_words2(const uint64_t* maps, int par, long i, long step, long nwords, uint64_t (&w)[2])
{
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const long wi = i + k * step < nwords ? i + k * step : i;
        w[k] = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(maps) + 2 * wi + par, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (i + step >= nwords) w[1] = 0;
    return true;
}

}  // namespace

}  // namespace cb
