// Fused back end, float32 and bfloat16, gathering from the channel-last shadow of the input state (Sec. III-A, last
// three processing steps in one kernel, like cb_fused_f32.hip).  The shadow holds the C values of a pixel side by
// side, so a filter tap of a listed pixel is C contiguous elements: fully coalesced 16-byte loads, no chunk table.
//
// Work item = BN listed columns x BM output channels x all of K; four wavefronts, WGM x WGN, each
// (16*TM) x (16*TN).  K is walked tap-major, k' = (j*kw + i)*Cs + c (Cs: the channels of a pixel of the shadow, C rounded up to
// whole 16-byte pieces), in groups of 32 (one step of v_mfma_f32_16x16x32_bf16), UKG groups = one stage.  Where Cs is a power of
// two (P2) a piece finds its tap by shifts; elsewhere the stage's first tap comes from one multiplication on the scalar unit, and a piece is
// in the tap of the stage's first value, dt taps on, or one further (cl_piece; two compares and adds a stage more).
//   B operand: a thread fetches 16-byte pieces of a column (consecutive lanes: consecutive pieces) and stores them to
//     LDS, [column][k], column pitch 4 mod 32 words (128 float32 columns: 20), so that the 16-byte fragment reads of eight
//     neighbouring columns cover all 32 banks.  Two stage buffers alternate; stage u+1 is stored and a later one requested between
//     the MFMAs of stage u (SPREAD) or ahead of them, one barrier per stage.  Narrow tiles, whose MFMAs are short, take long stages (the same
//     number of loads in flight whatever the tile width) and keep two of them in flight (GD).
//   A operand: packed in MFMA fragment order at layer creation, read from L2 into a ring of D groups of registers,
//     refilled as soon as a group's MFMAs are issued.
// The grid is persistent; N is read from device memory; each XCD takes a contiguous range of column tiles.
//
// float32 runs on the bfloat16 matrix cores as well.  A float32 product on v_mfma_f32_16x16x4_f32 costs sixteen
// times the matrix-core time of a bfloat16 one, and float32 layers were bound by exactly that (256 -> 256, 3x3, every
// output of 92x164: 166 us with or without the gather, the filter loads and the output stores).  Both operands are
// split into three bfloat16 terms, x * 2^24 = h + m + l, each the round-to-nearest bfloat16 of what the terms before it
// left over.  24 significant bits fit 3 x 8, and 2^24 in front keeps the last bit of float32's smallest numbers (2^-149) inside
// bfloat16's normal range, so the split is exact for every value below 2^104.  The six products down to 2^-16 of the
// leading one,
//     h*h + (h*m + m*h) + (h*l + m*m + l*h),
// are accumulated in float32: 6/16 of the matrix-core time.  What is left out (m*l, l*m, l*l) is below 2^-24 of the
// product; the sum over K is rounded once per 32 products instead of up to 32 times (TWO and GROUPED below).  Error against float64 over
// whole layers, float32 instruction / now: 64 -> 64 3x3 4.4e-7 / 1.3e-7, 128 -> 128 3x3 5.7e-7 / 1.3e-7, 256 -> 256 3x3 8.1e-7 /
// 1.7e-7.  The epilogue takes the 2^48 out again, exactly, together with the bias.  (Without the 2^24, values below 2^-110 lost
// their last term: 4e-6 of the result at 2^-116, 1e-3 at 2^-124.)
// The terms of an infinity, a NaN or a value of 2^104 and more do not add up to it, and sums beyond 2^80 overflow; any
// such makes the accumulated sum non-finite, and the epilogue recomputes every non-finite sum in plain
// float32 from the state and the filter matrix (exact_tiles), so that infinities, NaNs and large numbers come out as they do
// in float32 arithmetic.
#pragma once
#include "cb_fused.h"
#include "cb_cl_rules.h"

#include <type_traits>

namespace cb {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

// in front of both operands of a float32 product, and what takes them out of a sum of products
constexpr float SPLIT_SCALE = 0x1p24f, SPLIT_UNSCALE = 0x1p-48f;

// two neighbouring values (times SPLIT_SCALE) -> their three bfloat16 terms, packed
__device__ __forceinline__ void split2(float a, float b, unsigned& h, unsigned& m, unsigned& l)
{
    a *= SPLIT_SCALE;
    b *= SPLIT_SCALE;
    h = __builtin_bit_cast(unsigned, __builtin_convertvector(floatx2{a, b}, bf16x2));
    a -= __uint_as_float(h << 16);
    b -= __uint_as_float(h & 0xFFFF0000u);
    m = __builtin_bit_cast(unsigned, __builtin_convertvector(floatx2{a, b}, bf16x2));
    a -= __uint_as_float(m << 16);
    b -= __uint_as_float(m & 0xFFFF0000u);
    l = __builtin_bit_cast(unsigned, __builtin_convertvector(floatx2{a, b}, bf16x2));
}

// bits max(0, -o) .. min(k, size - o) - 1: which of a filter's k rows (columns), the first at o, lie inside the image
__device__ __forceinline__ unsigned taps_within(int o, int k, int size)
{
    const int lo = o < 0 ? -o : 0, hi = size - o < k ? size - o : k;
    return hi > lo ? ((1u << hi) - 1u) & ~((1u << lo) - 1u) : 0u;
}

// Sums whose split came out non-finite, in plain float32: TM 16 x 16 tiles of outputs on v_mfma_f32_16x16x4_f32, lane l16 =
// listed pixel q (-1: none) and filter row m + 16 * a (the wavefront's row tile at + a of krsrc).  A lane holds eight
// consecutive k' of a k-group: of the shadow as they are, of the filter matrix as the sum of its terms, which is the scaled
// filter value again; where it is not finite the value itself is fetched (KT: the filter matrix transposed, row (c*kh + j)*kw + i).
// A padding tap is a zero that takes part: zero times an infinite filter value is no number.
// Bound by the latency of its loads (few such sums) or the float32 matrix instruction (many).  Full updates, us, finite / one NaN /
// every value infinite: 64 -> 64, 3x3, 480x640 227 / 258 / 669, 256 -> 256, 3x3, 92x164 120 / 173 / 410.  A lane that walks K by itself
// for each of its sums took 547 / 28 100 and 2 606 / 16 960 for the latter two; a kernel on the float32 instruction throughout 330 and 180 for each.
template <int TM, bool P2>
__device__ __forceinline__ void exact_tiles(const Geom& g, const ClDiv& div, const __amdgpu_buffer_rsrc_t srsrc, const __amdgpu_buffer_rsrc_t krsrc,
                                            const float* __restrict__ KT, int nkg, int at, int lane, int q, int m, floatx4 (&sum)[TM])
{
    constexpr int U = P2 ? 2 : 1;                 // k-groups in flight (nkg is even; one without shifts: the second spilled registers of the whole kernel)
    const int lq = lane >> 4;
    const int lc = 31 - __builtin_clz((unsigned)g.Cs);       // (P2)
    const unsigned taps = (unsigned)(g.kh * g.kw);
    auto tap_of = [&](unsigned k) { return P2 ? k >> lc : cl_tap(div, k); };
    auto channel_of = [&](unsigned k, unsigned tap) { return P2 ? k & (unsigned)(g.Cs - 1) : k - tap * (unsigned)g.Cs; };
    auto pixels = [&](unsigned n) { return P2 ? n << lc : n * (unsigned)g.Cs; };
    const int qq = q < 0 ? 0 : q;
    const int yo = cl_row(div, qq, g.Wo);
    const int y0 = yo * g.s - g.p, x0 = (qq - yo * g.Wo) * g.s - g.p;
    const unsigned okr = q < 0 ? 0u : taps_within(y0, g.kh, g.H), okc = taps_within(x0, g.kw, g.W);
    const unsigned base = pixels((unsigned)(y0 * g.W + x0));
#pragma unroll
    for (int a = 0; a < TM; ++a) sum[a] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int kg = 0; kg < nkg; kg += U) {
        uint4 b[U][2], w[U][TM][3];
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const unsigned k = (unsigned)(32 * (kg + u) + 8 * lq + 4 * h), tap = tap_of(k);
                const unsigned j = (tap * div.inv_kw) >> 16, i = tap - j * (unsigned)g.kw;
                const bool in = (((okr >> (j < 31u ? j : 31u)) & (okc >> i)) & 1u) != 0u;
                const unsigned off = (base + pixels(j * (unsigned)g.W + i) + channel_of(k, tap)) * 4u;
                b[u][h] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(srsrc, (int)(in ? off : 0xFFFFFFF0u), 0, 0));
            }
#pragma unroll
            for (int a = 0; a < TM; ++a)
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    w[u][a][e] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(
                        krsrc, lane * 16 + e * 1024, (int)((unsigned)((at + a) * nkg + kg + u) * 3072u), 0));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float x[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = __uint_as_float(reinterpret_cast<const unsigned*>(&b[u][e >> 2])[e & 3]);
#pragma unroll
            for (int a = 0; a < TM; ++a) {
                float v[8];
                bool odd = false;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    auto term = [&](int t) {
                        const unsigned p = reinterpret_cast<const unsigned*>(&w[u][a][t])[e >> 1];
                        return __uint_as_float(e & 1 ? p & 0xFFFF0000u : p << 16);
                    };
                    v[e] = (term(0) + (term(1) + term(2))) * (1.f / SPLIT_SCALE);
                    odd |= !(fabsf(v[e]) < __builtin_inff());
                }
                if (__ballot(odd)) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const unsigned k = (unsigned)(32 * (kg + u) + 8 * lq + e), tap = tap_of(k), c = channel_of(k, tap);
                        if (!(fabsf(v[e]) < __builtin_inff())) v[e] = KT[((size_t)c * taps + tap) * g.Opad + m + 16 * a];
                    }
                }
#pragma unroll
                for (int e = 0; e < 8; ++e) sum[a] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[e], x[e], sum[a], 0, 0, 0);
            }
        }
    }
}

// k-groups per stage for a tile of bn columns (float32: 1 / 2 / 4 from 128 / 64 / 32 columns on).  Longer stages mean fewer
// barriers, shorter ones less padding of K and an earlier first MFMA.  bfloat16, twice as long: 64 -> 64 at 307 200
// listed pixels 70 against 50 us, 32 -> 32 43 against 28 us.
// (wgk: wavefronts that share a tile's K; each takes every wgk-th group of a stage)
template <typename T> __host__ __device__ constexpr int cl_groups(int bn, int wgk = 1)
{
    if (wgk > 1) return sizeof(T) == 4 ? 8 : 16;
    return sizeof(T) == 4 ? (bn >= 128 ? 1 : bn == 64 ? 2 : 4) : (bn >= 128 ? 2 : bn == 64 ? 4 : 8);
}
// bytes per column of a stage buffer, dynamic LDS (two buffers and the listed pixels; float32 three, bfloat16 four workgroups in 160 KB)
template <typename T> __host__ __device__ constexpr unsigned cl_pitch(int bn, int wgk = 1)
{
    return (unsigned)cl_groups<T>(bn, wgk) * (sizeof(T) == 4 ? 192u : 64u) + 16u;
}
template <typename T> __host__ __device__ constexpr unsigned cl_lds(int bn, int wgk = 1) { return 2u * (unsigned)bn * cl_pitch<T>(bn, wgk) + 4u * (unsigned)bn; }
constexpr unsigned CL_LDS_F32 = cl_lds<float>(128), CL_LDS_BF16 = cl_lds<uint16_t>(128);
static_assert(3 * CL_LDS_F32 <= 163840 && cl_lds<float>(64) <= CL_LDS_F32 && cl_lds<float>(32) <= CL_LDS_F32 && cl_lds<float>(16) <= CL_LDS_F32 &&
              4 * CL_LDS_BF16 <= 163840 && cl_lds<uint16_t>(64) <= CL_LDS_BF16 && cl_lds<uint16_t>(32) <= CL_LDS_BF16 &&
              cl_lds<uint16_t>(16) <= CL_LDS_BF16 && cl_lds<float>(16, 4) <= CL_LDS_F32 && cl_lds<uint16_t>(16, 4) <= CL_LDS_BF16,
              "the widest tile takes the most LDS");

// SPLIT: a tile's K is divided into `parts` ranges of stages, an item each.  An item leaves its sums in the workspace and counts itself; the
// tile's last one adds them up, in the order of K, and writes the outputs.
struct ClSplit { float* ws; int* count; unsigned parts; };
template <typename T, bool P2, int FAR, int WGM, int WGN, int TM, int TN, int WGK = 1, bool SPLIT = false>
__device__ __forceinline__ void fused_cl_body(const Geom& g, const ClDiv& div, const T* __restrict__ S2,
                                                 const int32_t* __restrict__ idx, const int N,
                                                 const uint4* __restrict__ KF, const float* __restrict__ KT,
                                                 const float* __restrict__ bias, int relu, T* __restrict__ OUT,
                                                 T* __restrict__ OUT2, const unsigned bx, const unsigned gx, const ClSplit& split = ClSplit())
{
    constexpr bool F32 = sizeof(T) == 4;
    constexpr int TERMS = F32 ? 3 : 1;           // bfloat16 terms per value
    constexpr int EPV = 16 / (int)sizeof(T);     // elements per 16-byte piece
    constexpr unsigned ESZ = (unsigned)sizeof(T);
    static_assert(WGM * WGN * WGK == 4, "four wavefronts per workgroup");
    constexpr int BM = 16 * TM * WGM, BN = 16 * TN * WGN;
    constexpr int UKG = cl_groups<T>(BN, WGK);   // k-groups of 32 per stage
    constexpr int UKW = UKG / WGK;               // ... of one wavefront
    constexpr int UK = 32 * UKG;
    constexpr int PPC = UK / EPV;                // 16-byte pieces of a column in a stage
    constexpr int CPP = 256 / PPC;               // columns one round of loads covers
    constexpr int NP = BN / CPP;                 // loads per thread and stage
    static_assert(PPC <= 64 && NP * CPP == BN, "pieces come out even");
    // k-groups of filter fragments in flight: an L2 latency's worth of MFMAs, as far as the registers go
    constexpr int DMAX = F32 ? (TM == 1 ? 4 : 2)
                          : (TM * TN <= 2 ? 8 : TM * TN <= 8 ? 4 : 2);
    constexpr int D = DMAX < 4 * UKW ? DMAX : 4 * UKW;
    constexpr int GD = F32 && TM * TN <= 2 ? 2 : 1;     // stages of gathered pieces in flight
    // stages per round of the stage loop: ring slot and register set are compile-time indexes
    constexpr int UU = D / UKW > GD ? D / UKW : GD;
    static_assert(UU * UKW % D == 0 && UU % GD == 0, "a round of stages is whole rings");
    constexpr unsigned PITCH = cl_pitch<T>(BN, WGK), BUF = BN * PITCH;
    constexpr unsigned PLANE = UKG * 64u;        // bytes of one term of a column
    // the largest tile has no registers for what can be fetched when it is used: the next tile's pixels, the bias, a longer ring
    constexpr bool LEAN = TM * TN > 8;
    // Column fragments of a wavefront and stage, and how many of them are in registers.  SPREAD: the next stages' pieces are passed on between the products of
    // this one.  A narrow tile has one or two wavefronts on a SIMD, and what one does not overlap itself is not overlapped: with one fragment ahead and
    // everything else in front of the products a k-group of 64 x 32 bfloat16 tiles took 210 cycles, for 32 of matrix instructions and 96 of L1, whether its loads
    // hit or missed.  Frames, us, before / now: 512 -> 512 3x3 46x82 10 % bfloat16 42.4 / 39.5, 256 -> 256 3x3 92x164 30.2 / 29.2, bfloat16 10 % 28.1 / 26.9, 32 -> 32 9x9 at
    // 240x320 29.9 / 28.6, a full update of 256 -> 256 92x164 107.0 / 102.5.  Wider bfloat16 tiles have the wavefronts and not the registers (128 x 128 spread: 458 / 544).
    constexpr bool SPREAD = F32 ? TM * TN <= (P2 ? 8 : 4) : TM * TN <= 2 && WGK == 1;
    constexpr int NF = UKW * TN, BR = !F32 && SPREAD ? 4 : 2;
    // float32: what rounds a sum is every product that is added to it.  TWO: the five small ones of a group are a second chain, where there are registers for its sums.  GROUPED: the six
    // of a group are summed from zero and added at once; 4 vector additions, 16 cycles, for 96 of matrix instructions.  Relative errors of whole layers against float64, one chain of six / so:
    // 128 -> 128 3x3 5.3e-7 / 1.3e-7, 256 -> 256 3x3 7.3e-7 / 1.7e-7, 64 -> 256 7x7 8.7e-7 / 1.9e-7, 32 -> 32 3x3 2.5e-7 / 0.9e-7.  us: full update of 256 -> 256 92x164 104.9 / 108.8, of 64 -> 256 7x7
    // 120x160 172.3 / 179.6, of 64 -> 64 480x640 197.1 / 198.5, 128 -> 128 1080p 2 % changed 456.0 / 460.3, five-layer net 116.8 / 116.5.
    constexpr bool TWO = TM * TN < 4 || (F32 && TM * TN == 4), GROUPED = F32 && !TWO;
    extern __shared__ uint4 dyn_lds4[];          // two stage buffers, then the listed pixel of every column
    char* const Bs = reinterpret_cast<char*>(dyn_lds4);
    int* const qs = reinterpret_cast<int*>(Bs + 2 * BUF);
    float* const bs = reinterpret_cast<float*>(qs + BN + 4);      // (GROUPED: the tile's bias, for which there are no registers; behind it and the pixels SPLIT has a word)
    static_assert(!GROUPED || 2 * BUF + 4 * (BN + 4 + BM) <= cl_lds<T>(128), "room for a tile's bias");

    const int nkg = F32 ? (g.Cs * g.kh * g.kw + 63) / 64 * 2 : (g.Cs * g.kh * g.kw + 127) / 128 * 4;       // k-groups of the packed filter matrix
    const int stages = (nkg + UKG - 1) / UKG;
    const unsigned parts = SPLIT ? split.parts : 1u;
    const int lc = 31 - __builtin_clz((unsigned)g.Cs);       // (P2)
    auto pixels = [&](unsigned n) { return P2 ? n << lc : n * (unsigned)g.Cs; };
    const __amdgpu_buffer_rsrc_t srsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<T*>(S2), 0, (int)((unsigned)g.Cs * (unsigned)g.P * ESZ), 0x00020000);
    constexpr unsigned NOWHERE = 0xFFFFFFF0u;
    // tiles: every XCD (workgroup number mod 8) walks its own range of column tiles, all row tiles of one column tile in
    // turn; with filters that half an XCD's L2 does not hold (FAR) the XCDs are 2, 4 or 8 groups with a range of the row tiles each
    // (cl_xcd_rows).  (32 bits: the outputs of 2^31 such tiles would not fit any memory.)
    const unsigned NT = ((unsigned)N + BN - 1u) / BN;
    const unsigned MT = ((unsigned)g.O + BM - 1u) / BM;
    const unsigned lx = FAR ? cl_xcd_rows(MT, NT, parts, cl_filter_kb(g.O, (unsigned)nkg, F32), cl_pixel_kb((unsigned)N, (unsigned)g.Cs, ESZ)) : 0u;
    const unsigned MTX = FAR ? (MT + (1u << lx) - 1u) >> lx : MT, mt0 = FAR ? (bx & ((1u << lx) - 1u)) * MTX : 0u;
    const unsigned per_xcd = FAR ? (NT + (8u >> lx) - 1u) >> (3u - lx) : (NT + 7u) / 8u, total = per_xcd * MTX * parts;
    const unsigned xcd0 = (FAR ? (bx & 7u) >> lx : bx & 7u) * per_xcd;

    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int wk = __builtin_amdgcn_readfirstlane(wv % WGK);
    const int wm = wv / WGK / WGN, wn = wv / WGK % WGN;
    const int wm_s = __builtin_amdgcn_readfirstlane(wm);
    const int l16 = lane & 15, lq = lane >> 4;
    const int gc = tid / PPC, ch = tid % PPC;    // first column of this thread, its piece of a stage
    const int dt = P2 ? (EPV * ch) >> lc : (int)cl_tap(div, (unsigned)(EPV * ch)), cl = P2 ? (EPV * ch) & (g.Cs - 1) : EPV * ch - dt * g.Cs;

    // Of the NP columns that a column group of lanes fetches, lane ch has the pixel of column ch % NP, and works out what the others need of it (one column after
    // the other in every lane took 0.3 us a tile)
    static_assert(PPC >= NP && (NP & (NP - 1)) == 0, "a lane for each column");
    // The thread's number as a value that the compiler does not know, so that what follows from it is worked out again for each tile, ahead of and behind its stages, and not held
    // over them, for which there are no registers: with such numbers held 14 of the 16 float32 kernels spilled 1 - 12 of them (a reload ahead of a tile's first stage waits for
    // every load in flight), now none, and bfloat16's with 128 x 128 tiles 13 - 21, now 7 - 12.  Frames are the same within 1 %.
    auto thread_again = [&]() {
        int t = (int)threadIdx.x;
        asm volatile("" : "+v"(t));
        return t;
    };
    auto column_of = [&](int t) { return t / PPC + CPP * (t % PPC & (NP - 1)); };
    auto fetch_q = [&](unsigned u, int col) {
        const unsigned n = (xcd0 + (SPLIT ? u / parts : u) / MTX) * BN + col;
        const int q = idx[n < (unsigned)N ? n : (unsigned)N - 1u];
        return u < total && n < (unsigned)N ? q : -1;
    };
    int qnext = -1;
    if constexpr (!LEAN) qnext = fetch_q(bx >> 3, column_of(tid));

    for (unsigned uq = bx >> 3; uq < total; uq += gx >> 3) {
        const unsigned ut = SPLIT ? uq / parts : uq;
        const int mt = (int)(FAR ? mt0 + ut % MTX : ut % MTX);
        const unsigned nt = xcd0 + ut / MTX;
        // this item's stages: nunits from u0 on
        const unsigned part = SPLIT ? uq % parts : 0u;
        const int u0 = SPLIT ? (int)(part * (unsigned)stages / parts) : 0;
        const int nunits = SPLIT ? (int)((part + 1u) * (unsigned)stages / parts) - u0 : stages;
        const int t0 = thread_again(), mycol = column_of(t0);
        int q = qnext;
        if constexpr (LEAN) q = fetch_q(uq, mycol);
        else qnext = fetch_q(uq + (gx >> 3), mycol);
        if (nt >= NT || (FAR && (unsigned)mt >= MT)) continue;
        const int m0 = mt * BM;

        // ring of filter fragments: [k-group mod D][row tile][term].  The resource covers this tile's rows.
        const __amdgpu_buffer_rsrc_t krsrc = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint4*>(KF) + (size_t)(m0 >> 4) * nkg * (TERMS * 64), 0,
            (int)((unsigned)(BM / 16) * (unsigned)nkg * (TERMS * 1024u)), 0x00020000);
        uint4 areg[D][TM][TERMS];
        auto aload = [&](int kg, uint4 (&dst)[TM][TERMS]) {
            const int kc = kg < nkg ? kg : nkg - 1;
#pragma unroll
            for (int a = 0; a < TM; ++a) {
                const unsigned soff = (unsigned)((wm_s * TM + a) * nkg + kc) * (TERMS * 1024u);
#pragma unroll
                for (int e = 0; e < TERMS; ++e)
                    dst[a][e] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(krsrc, lane * 16 + e * 1024, (int)soff, 0));
            }
        };

        // per column: which filter rows and columns lie inside the image (all clear for a column without a pixel), and the
        // byte offset of the top-left tap's channel cl in the shadow (it may wrap below zero at the border: only
        // taps inside are fetched, and for those the sum is a valid offset again)
        unsigned outr[NP], outc[NP], base[NP];
        {
            const bool colv = q >= 0;
            const int qq = colv ? q : 0;
            const int yo = cl_row(div, qq, g.Wo);
            const int xo = qq - yo * g.Wo;
            const int y0 = yo * g.s - g.p, x0 = xo * g.s - g.p;
            const unsigned r = ~(colv ? taps_within(y0, g.kh, g.H) : 0u), c = ~taps_within(x0, g.kw, g.W), b = pixels((unsigned)(y0 * g.W + x0)) * ESZ;
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const int from = (t0 & 63 & ~(PPC - 1)) + p;      // (PPC: up to a wavefront)
                outr[p] = (unsigned)__shfl((int)r, from);
                outc[p] = (unsigned)__shfl((int)c, from);
                base[p] = (unsigned)__shfl((int)b, from) + (unsigned)cl * ESZ;
            }
        }

        uint4 breg[GD][NP];
        // stage u's piece of every column: its filter row and column, its offset
        struct Piece { unsigned j, i, off; };
        auto piece_of = [&](int u) {
            const unsigned kb = (unsigned)(SPLIT ? u0 + u : u) * (unsigned)UK;
            unsigned tap, coff;                  // the piece's tap, its channel less cl
            if constexpr (P2) { tap = (kb >> lc) + (unsigned)dt; coff = kb & (unsigned)(g.Cs - 1); }
            else cl_piece(div, (unsigned)g.Cs, kb, (unsigned)dt, (unsigned)cl, tap, coff);
            const unsigned j = (tap * div.inv_kw) >> 16, i = tap - j * (unsigned)g.kw;
            // (rows that pad K have j >= kh, whose bit is set, as bit 31 is for any j beyond it: kh, kw <= 31)
            return Piece{j < 31u ? j : 31u, i, (pixels(j * (unsigned)g.W + i) + coff) * ESZ};
        };
        // (all ones for a tap outside the image: the offset is NOWHERE then, base and off are multiples of 16)
        auto gload = [&](const Piece& w, int p) {
            const unsigned out = (unsigned)(__builtin_amdgcn_sbfe((int)outr[p], w.j, 1u) | __builtin_amdgcn_sbfe((int)outc[p], w.i, 1u));
            return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(srsrc, (int)((out & NOWHERE) | (base[p] + w.off)), 0, 0));
        };
        auto lds_store = [&](int buf, int p, const uint4& v) {
            char* dst = Bs + buf * BUF + gc * PITCH + (F32 ? 8 : 16) * ch;
            if constexpr (F32) {
                uint2 h, m, l;
                split2(__uint_as_float(v.x), __uint_as_float(v.y), h.x, m.x, l.x);
                split2(__uint_as_float(v.z), __uint_as_float(v.w), h.y, m.y, l.y);
                *reinterpret_cast<uint2*>(dst + CPP * p * PITCH) = h;
                *reinterpret_cast<uint2*>(dst + CPP * p * PITCH + PLANE) = m;
                *reinterpret_cast<uint2*>(dst + CPP * p * PITCH + 2 * PLANE) = l;
            } else
                *reinterpret_cast<uint4*>(dst + CPP * p * PITCH) = v;
        };

        floatx4 acc[TM][TN], acc1[TM][TN];         // (acc1: unused unless TWO)
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int b = 0; b < TN; ++b) {
                acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
                acc1[a][b] = acc[a][b];
            }

        // (the loads in flight at the stage loop's entry are in the order of those in flight at its back edge: where
        // the two differ the compiler waits for the longer of the two queues)
        auto gather = [&](int u, uint4 (&dst)[NP]) {
            const Piece w = piece_of(u);
#pragma unroll
            for (int p = 0; p < NP; ++p) dst[p] = gload(w, p);
        };
        gather(0, breg[0]);
        if constexpr (GD == 2) {
            gather(1, breg[1]);
#pragma unroll
            for (int s = 0; s < D; ++s) aload((SPLIT ? u0 * UKG : 0) + s * WGK + wk, areg[s]);
        }
        float bv[TM][4];                          // bias of this wavefront's rows
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = m0 + (wm * TM + a) * 16 + (t0 & 63) / 16 * 4 + r;
                bv[a][r] = LEAN || GROUPED ? 0.f : bias[m < g.O ? m : g.O - 1];
            }
        float bias_of = 0.f;
        if constexpr (GROUPED) bias_of = bias[m0 + t0 % BM < g.O ? m0 + t0 % BM : g.O - 1];
        __syncthreads();                          // the previous tile has read its last stage, its qs and its bias
        if constexpr (GROUPED) {
            static_assert(BM <= 256, "a thread for each row");
            if (t0 < BM) bs[t0] = bias_of;
        }
        if (ch < NP) qs[mycol] = q;
#pragma unroll
        for (int p = 0; p < NP; ++p) lds_store(0, p, breg[0][p]);
        gather(GD, breg[0]);
        if constexpr (GD == 1) {
#pragma unroll
            for (int s = 0; s < D; ++s) aload((SPLIT ? u0 * UKG : 0) + s * WGK + wk, areg[s]);
        }
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();

        const char* const Bw = Bs + (wn * TN * 16 + l16) * PITCH + lq * 16;
        // SI: stage modulo UU
        auto stage = [&](int u, auto si) {
            constexpr int SI = decltype(si)::value;
            constexpr int S0 = SI * UKW % D;      // ring slot of the stage's first k-group
            const int cur = u & 1;
            const char* const Bu = Bw + cur * BUF;
            // ring of column fragments, f = kgi * TN + b (those of k-groups behind the last are read, and not used)
            uint4 bfr[BR][TERMS];
            auto bload = [&](int f) {
#pragma unroll
                for (int e = 0; e < TERMS; ++e)
                    bfr[f % BR][e] = *reinterpret_cast<const uint4*>(Bu + (f % TN) * 16 * PITCH + e * PLANE + (f / TN * WGK + wk) * 64);
            };
#pragma unroll
            for (int f = 0; f + 1 < BR && f < NF; ++f) bload(f);
            // stage u+1 goes into the buffer that stage u-1 was read from; stage u+1+GD is requested: piece by piece between the products
            const Piece w = piece_of(u + 1 + GD);
            auto pass_on = [&](int p) {
                if (u + 1 < nunits) lds_store(cur ^ 1, p, breg[(SI + 1) % GD][p]);
                breg[(SI + 1) % GD][p] = gload(w, p);
            };
            if constexpr (!SPREAD) {
                if (u + 1 < nunits) {
#pragma unroll
                    for (int p = 0; p < NP; ++p) lds_store(cur ^ 1, p, breg[(SI + 1) % GD][p]);
                }
#pragma unroll
                for (int p = 0; p < NP; ++p) breg[(SI + 1) % GD][p] = gload(w, p);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int kgi = 0; kgi < UKW; ++kgi) {
                const int kg = (SPLIT ? u0 + u : u) * UKG + kgi * WGK + wk;
                // the last stage may be short (whole pairs / fours of k-groups)
                if ((WGK > 1 || (kgi > 0 && kgi % (F32 ? 2 : 4) == 0)) && kg >= nkg) break;
                uint4 (&af)[TM][TERMS] = areg[(S0 + kgi) % D];
#pragma unroll
                for (int b = 0; b < TN; ++b) {
                    const int f = kgi * TN + b;
                    if (f + BR - 1 < NF) bload(f + BR - 1);
                    auto mul = [&](int ea, int eb, floatx4 (&d)[TM][TN]) {
#pragma unroll
                        for (int a = 0; a < TM; ++a)
                            d[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, af[a][ea]),
                                                                              __builtin_bit_cast(bf16x8, bfr[f % BR][eb]), d[a][b], 0, 0, 0);
                    };
                    if constexpr (GROUPED) {
                        floatx4 t[TM];
                        auto term = [&](int ea, int eb, bool first) {
#pragma unroll
                            for (int a = 0; a < TM; ++a)
                                t[a] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, af[a][ea]), __builtin_bit_cast(bf16x8, bfr[f % BR][eb]),
                                                                               first ? floatx4{0.f, 0.f, 0.f, 0.f} : t[a], 0, 0, 0);
                        };
                        term(2, 0, true); term(1, 1, false); term(0, 2, false); term(1, 0, false); term(0, 1, false); term(0, 0, false);
#pragma unroll
                        for (int a = 0; a < TM; ++a) {
                            acc[a][b] += t[a];
                            asm volatile("" : "+v"(acc[a][b]));       // (here: moved to the end of the stage all additions' operands are held, and 66 - 126 registers spill)
                        }
                    } else if constexpr (F32) {
                        // smallest terms first; a chain of their own where a wavefront has few tiles
                        floatx4 (&rest)[TM][TN] = TWO ? acc1 : acc;
                        mul(2, 0, rest); mul(1, 1, rest); mul(0, 2, rest); mul(1, 0, rest); mul(0, 1, rest);
                        mul(0, 0, acc);
                    } else
                        mul(0, 0, TWO && (kgi & 1) ? acc1 : acc);
                    if constexpr (SPREAD) {
#pragma unroll
                        for (int p = 0; p < NP; ++p)
                            if (p * NF / NP == f) pass_on(p);
                    }
                }
                aload(kg + D * WGK, af);
                __builtin_amdgcn_sched_barrier(0);
            }
            __syncthreads();
        };
        for (int u = 0; u < nunits; u += UU) {
            stage(u, std::integral_constant<int, 0>());
            if constexpr (UU >= 2) if (u + 1 < nunits) stage(u + 1, std::integral_constant<int, 1>());
            if constexpr (UU >= 4) {
                if (u + 2 < nunits) stage(u + 2, std::integral_constant<int, 2>());
                if (u + 3 < nunits) stage(u + 3, std::integral_constant<int, 3>());
            }
            static_assert(UU == 1 || UU == 2 || UU == 4, "stages per round");
        }

        const int lane_o = thread_again() & 63, l16o = lane_o & 15, lqo = lane_o >> 4;
        if (TWO) {
#pragma unroll
            for (int a = 0; a < TM; ++a)
#pragma unroll
                for (int b = 0; b < TN; ++b) acc[a][b] += acc1[a][b];
        }
        if constexpr (WGK > 1) {
            // the partial sums of the other wavefronts, through the (now free) stage buffers, added in their order
            float* const red = reinterpret_cast<float*>(Bs) + lane_o;
            constexpr int PER = TM * TN * 4 * 64;
            static_assert((unsigned)(4 * PER) * 4u <= 2u * BUF, "partial sums fit the stage buffers");
            if (wk) {
#pragma unroll
                for (int a = 0; a < TM; ++a)
#pragma unroll
                    for (int b = 0; b < TN; ++b)
#pragma unroll
                        for (int r = 0; r < 4; ++r) red[wv * PER + ((a * TN + b) * 4 + r) * 64] = acc[a][b][r];
            }
            __syncthreads();
            if (wk) continue;
#pragma unroll
            for (int w = 1; w < WGK; ++w)
#pragma unroll
                for (int a = 0; a < TM; ++a)
#pragma unroll
                    for (int b = 0; b < TN; ++b)
#pragma unroll
                        for (int r = 0; r < 4; ++r) acc[a][b][r] += red[(wv + w) * PER + ((a * TN + b) * 4 + r) * 64];
        }
        if constexpr (SPLIT) {
            static_assert(WGK == 1, "parts are whole workgroups");
            // Written through to where every XCD sees them; the count follows when all of the workgroup's are there.
            const unsigned tile = nt * MT + (unsigned)mt;
            typedef unsigned long long u64;
            u64* const mine = reinterpret_cast<u64*>(split.ws) + (size_t)(tile * parts) * (BM * BN / 2) + tid;
            auto word = [&](const floatx4& v, int h) { return (u64)__float_as_uint(v[2 * h]) | (u64)__float_as_uint(v[2 * h + 1]) << 32; };
#pragma unroll
            for (int a = 0; a < TM; ++a)
#pragma unroll
                for (int b = 0; b < TN; ++b)
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        __hip_atomic_store(mine + part * (BM * BN / 2) + ((a * TN + b) * 2 + h) * 256, word(acc[a][b], h), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
            asm volatile("" ::: "memory");
            int* const s_last = qs + BN;
            __syncthreads();
            if (tid == 0) *s_last = (unsigned)__hip_atomic_fetch_add(split.count + tile, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == parts - 1u;
            __syncthreads();
            if (!*s_last) continue;
            if (tid == 0) split.count[tile] = 0;  // for the next launch
            floatx4 sum[TM][TN];
#pragma unroll
            for (int a = 0; a < TM; ++a)
#pragma unroll
                for (int b = 0; b < TN; ++b) sum[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
            // (a batch of parts in flight: one after the other they take a round trip to memory each)
            constexpr int PB = TM * TN <= 4 ? 4 : 2;
#pragma unroll 1
            for (unsigned p0 = 0; p0 < parts; p0 += PB) {
                u64 w[PB][TM * TN * 2];
#pragma unroll
                for (int q = 0; q < PB; ++q)
#pragma unroll
                    for (int i = 0; i < TM * TN * 2; ++i) {
                        const unsigned p = p0 + q < parts ? p0 + q : part;
                        w[q][i] = __hip_atomic_load(mine + p * (BM * BN / 2) + i * 256, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
#pragma unroll
                for (int q = 0; q < PB; ++q)
                    if (p0 + q < parts)
#pragma unroll
                        for (int i = 0; i < TM * TN * 2; ++i) {
                            floatx4& d = sum[i / 2 / TN][i / 2 % TN];
                            d[2 * (i & 1)] += __uint_as_float((unsigned)w[q][i]);
                            d[2 * (i & 1) + 1] += __uint_as_float((unsigned)(w[q][i] >> 32));
                        }
            }
#pragma unroll
            for (int a = 0; a < TM; ++a)
#pragma unroll
                for (int b = 0; b < TN; ++b) acc[a][b] = sum[a][b];
        }
        if constexpr (GROUPED) {
#pragma unroll
            for (int a = 0; a < TM; ++a) {
                const floatx4 v = *reinterpret_cast<const floatx4*>(bs + (wm * TM + a) * 16 + lqo * 4);
#pragma unroll
                for (int r = 0; r < 4; ++r) bv[a][r] = v[r];
            }
        }
        if constexpr (LEAN) {
#pragma unroll
            for (int a = 0; a < TM; ++a)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int m = m0 + (wm * TM + a) * 16 + lqo * 4 + r;
                    bv[a][r] = bias[m < g.O ? m : g.O - 1];
                }
        }
        // output update: bias + ReLU, written at the listed pixels only
        unsigned long long bad = 0;               // float32: sums to recompute, bit (b*TM + a)*4 + r
        const int mw = m0 + wm_s * TM * 16;       // first row of this wavefront
        T* const orow = OUT + (size_t)(mw + lqo * 4) * g.Po;
        const bool whole = mw + 16 * TM <= g.O;
#pragma unroll
        for (int b = 0; b < TN; ++b) {
            const int qn = qs[(wn * TN + b) * 16 + l16o];
            if (qn < 0) continue;
            T* const o = orow + qn;
            auto rows = [&](bool all) {
#pragma unroll
                for (int a = 0; a < TM; ++a) {
                    const int mb = mw + a * 16 + lqo * 4;
                    float v4[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        float v = F32 ? fmaf(acc[a][b][r], SPLIT_UNSCALE, bv[a][r]) : acc[a][b][r] + bv[a][r];
                        if (F32 && !(fabsf(acc[a][b][r]) < __builtin_inff()) && (all || mb + r < g.O)) bad |= 1ull << ((b * TM + a) * 4 + r);
                        if (relu) v = v > 0.f ? v : 0.f;
                        if (all || mb + r < g.O) st_out(o + (size_t)(a * 16 + r) * g.Po, v);
                        v4[r] = v;
                    }
                    // (a layer that keeps the pixel-major copy has a multiple of 16 output channels)
                    if (OUT2 && (all || mb < g.O)) st_out4(OUT2 + (size_t)qn * g.O + mb, v4);
                }
            };
            if (whole) rows(true);
            else rows(false);
        }
        if constexpr (F32) {
            if (__ballot(bad != 0ull))
#pragma unroll 1
                for (int b = 0; b < TN; ++b) {
                    const unsigned mine = (unsigned)(bad >> (4 * TM * b)) & ((1u << (4 * TM)) - 1u);
                    if (!__ballot(mine != 0u)) continue;
                    const int qn = qs[(wn * TN + b) * 16 + l16o];
                    floatx4 sum[TM];
                    exact_tiles<TM, P2>(g, div, srsrc, krsrc, KT, nkg, wm_s * TM, lane_o, qn, mw + l16o, sum);
#pragma unroll
                    for (int a = 0; a < TM; ++a)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (mine & (1u << (4 * a + r))) {
                                const int m = mw + a * 16 + lqo * 4 + r;
                                float v = sum[a][r] + bias[m];
                                if (relu) v = v > 0.f ? v : 0.f;
                                OUT[(size_t)m * g.Po + qn] = v;
                                if (OUT2) OUT2[(size_t)qn * g.O + m] = v;
                            }
                }
        }
    }
}

// The arguments of a launch, requested at once: left to itself the compiler asks for the count's address, the count, and, once that is known not to be zero, in two
// or three rounds for the rest.  With this and the pixels worked out by a lane each, frames, us: ten-layer trunk bfloat16 146.8 / 139.5, 64 -> 128 271x435 bfloat16
// 20.1 / 19.7, 48 -> 96 5x5 stride 2 241x323 26.3 / 25.7, 64 -> 32 240x320 21.1 / 20.2, 16 -> 16 1x1 368x656 15.3 / 14.8.
template <typename T>
__device__ __forceinline__ void hold_arguments(const Geom& g, const ClDiv& div, const T* S2, const int32_t* idx, const int* count, const uint4* KF, const float* KT, const float* bias, int relu,
                                               const T* OUT, const T* OUT2)
{
    asm volatile("" :: "s"(count), "s"(idx), "s"(S2), "s"(KF), "s"(bias), "s"(OUT), "s"(OUT2), "s"(relu), "s"(g.O), "s"(g.Cs), "s"(g.kh), "s"(g.kw), "s"(g.s), "s"(g.p), "s"(g.H),
                 "s"(g.W));
    asm volatile("" :: "s"(KT), "s"(g.Opad), "s"(g.Wo), "s"(g.P), "s"(g.Po), "s"(g.R), "s"(div.inv_wo), "s"(div.inv_kw), "s"(div.inv_cs));
}

// Workgroups of a launch.  (A constant: read from the launch's hidden arguments it lies beyond the kernel's own, on a line of its own, and was
// up to 0.3 us of a launch: ten-layer trunk at 368x656, bfloat16, 155.1 us a frame, 152.3 without it.)
constexpr unsigned CL_GRID = 1024;

// workgroup bx of gx
template <typename T, int SHAPE, bool P2, int FAR>
__device__ __forceinline__ void fused_cl_run(const Geom& g, const ClDiv& div, const T* __restrict__ S2, const int32_t* __restrict__ idx,
                                             const int* __restrict__ count, const uint4* __restrict__ KF, const float* __restrict__ KT,
                                             const float* __restrict__ bias, int relu, T* __restrict__ OUT, T* __restrict__ OUT2,
                                             const unsigned bx, const unsigned gx, float* ws, unsigned ws_bytes, int* kcount)
{
    hold_arguments(g, div, S2, idx, count, KF, KT, bias, relu, OUT, OUT2);
    const int N = *(const __attribute__((address_space(4))) int*)count;       // (a scalar load: nothing of this launch writes it)
    if (N <= 0) return;
    if constexpr (FAR == 2) {
        const unsigned sp = cl_split<sizeof(T) == 4>(N, g.O, ((unsigned)(g.Cs * g.kh * g.kw) + 31u) / 32u, ws_bytes);
        if (sp) {
            const ClSplit split{ws, kcount, sp & 15u};
            if (sp & 16u) fused_cl_body<T, P2, FAR, 4, 1, 2, 4, 1, true>(g, div, S2, idx, N, KF, KT, bias, relu, OUT, OUT2, bx, gx, split);
            else fused_cl_body<T, P2, FAR, 4, 1, 2, 2, 1, true>(g, div, S2, idx, N, KF, KT, bias, relu, OUT, OUT2, bx, gx, split);
            return;
        }
    }
#define CB_BODY(...) fused_cl_body<T, P2, FAR, __VA_ARGS__>(g, div, S2, idx, N, KF, KT, bias, relu, OUT, OUT2, bx, gx)
    // (the tiles of cb_cl_rules.h)
    cl_tile<sizeof(T) == 4, SHAPE>(N, g.O, g.Cs, g.kh * g.kw, g.R, [&](auto tile) __attribute__((always_inline)) {
        constexpr int t = decltype(tile)::value;
        static_assert(t < cl_tiles(SHAPE), "a tile of this instance");
        if constexpr (t == 0) CB_BODY(1, 1, 1, 1, 4);
        else if constexpr (SHAPE == 16) CB_BODY(1, 4, 1, t);
        else if constexpr (SHAPE == 32) CB_BODY(2, 2, 1, 1 << (t - 1));
        else if constexpr (SHAPE == 64 || t <= 2) CB_BODY(4, 1, 1, 1 << (t - 1));
        else if constexpr (t == 5) CB_BODY(4, 1, 2, 8);
        else CB_BODY(4, 1, 2, 1 << (t - 2));
    });
#undef CB_BODY
}

// (wavefronts per SIMD: as many as the widest tile's registers allow.  They are worth more than wider tiles: bfloat16, O > 64
// at 76 800 listed pixels 45 us with two, 40 us with four.)
template <typename T, int SHAPE, bool P2, int FAR>
__global__ __launch_bounds__(256, sizeof(T) == 2 ? 4 : 3) void fused_cl_kernel(Geom g, ClDiv div, const T* __restrict__ S2,
                                                          const int32_t* __restrict__ idx, const int* __restrict__ count,
                                                          const uint4* __restrict__ KF, const float* __restrict__ KT,
                                                          const float* __restrict__ bias, int relu,
                                                          T* __restrict__ OUT, T* __restrict__ OUT2, float* ws, unsigned ws_bytes, int* kcount)
{
    fused_cl_run<T, SHAPE, P2, FAR>(g, div, S2, idx, count, KF, KT, bias, relu, OUT, OUT2, blockIdx.x, CL_GRID, ws, ws_bytes, kcount);
}

// run(an integral constant: the kernel's instance) for a layer of this geometry; its arguments checked
template <typename T, typename FN>
hipError_t fused_cl_instance(const Geom& g, const FusedPlan& plan, FN&& run)
{
    if (!plan.cl || g.Cs % (16 / (int)sizeof(T)) != 0 || g.Cs < g.C || !cl_fits(g.Cs, g.kh * g.kw) || g.bf16 != (sizeof(T) == 2)) return hipErrorInvalidValue;
    switch (cl_shape(g.O, g.Po, sizeof(T) == 4)) {
        case 16: run(std::integral_constant<int, 16>()); break;
        case 32: run(std::integral_constant<int, 32>()); break;
        case 64: run(std::integral_constant<int, 64>()); break;
        case 129: if constexpr (sizeof(T) == 2) run(std::integral_constant<int, 129>()); break;
        default: run(std::integral_constant<int, 128>());
    }
    return hipGetLastError();
}
// FAR = 1: layers whose XCDs divide the row tiles among them; 2: which may divide K as well.  In instances of their own, since the few
// instructions more, and what they do to the allocation of scalar registers, cost the layers that use neither 0.2 - 0.7 us a launch (64 -> 128,
// 128 -> 128, bfloat16; 256 -> 256, 3x3, 92x164 23.6 / 24.4 us).
inline int fused_cl_far_mode(const Geom& g, const ClWork& work)
{
    return !fused_cl_far(g) ? 0 : work.bytes && cl_shape(g.O, g.Po, !g.bf16) == 128 ? 2 : 1;
}
template <typename T> constexpr unsigned cl_lds_bytes() { return sizeof(T) == 4 ? CL_LDS_F32 : CL_LDS_BF16; }

template <typename T>
hipError_t launch_fused_cl(const Geom& g, const FusedPlan& plan, const T* shadow, const int32_t* idx, const int* count,
                           const void* KF, const float* KT, const float* bias, int relu, T* OUT, T* OUT2, const ClWork& work, hipStream_t st, Tm tm)
{
    const ClDiv div = cl_div(g.Wo, g.Ho, g.kw, g.Cs);
    const bool p2 = (g.Cs & (g.Cs - 1)) == 0;
    return fused_cl_instance<T>(g, plan, [&](auto shape) {
        constexpr int SHAPE = decltype(shape)::value;
#define CB_CL(p, far) \
    CB_LAUNCH_LDS((fused_cl_kernel<T, SHAPE, p, far>), dim3(CL_GRID), dim3(256), cl_lds_bytes<T>(), st, tm, g, div, shadow, \
                  idx, count, (const uint4*)KF, KT, bias, relu, OUT, OUT2, work.ws, work.bytes, work.count)
        const int far = fused_cl_far_mode(g, work);
        if constexpr (SHAPE == 128)
            if (far == 2) {
                CB_CL(true, 2);
                return;
            }
        if constexpr (SHAPE >= 128)
            if (far) {
                CB_CL(true, 1);
                return;
            }
        if (p2) CB_CL(true, 0);
        else CB_CL(false, 0);
#undef CB_CL
    });
}

}  // namespace

}  // namespace cb
