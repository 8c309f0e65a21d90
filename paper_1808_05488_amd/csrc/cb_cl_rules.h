// Rules of the channel-last fused kernel (cb_fused_cl.h) that need no GPU: plain arithmetic on the geometry, usable
// from host code and kernels alike.
#pragma once

#include <type_traits>

#ifdef __HIPCC__
#define CB_HD __host__ __device__ __forceinline__
#else
#define CB_HD inline
#endif

namespace cb {

// Divisions by layer constants.  tap / kw = tap * inv_kw >> 16 for the few taps there are.  q / Wo = q * inv_wo >> 42
// with inv_wo = ceil(2^42 / Wo) (0: divide).  The quotient is exact while q * Wo < 2^42: q < 2^30 in every layer, so Wo < 2^12
// is enough.  The product lies below (q / Wo + 1) * 2^42 and has to fit 64 bits, which takes Ho <= 2^22.
// k / Cs = k * inv_cs >> 32 with inv_cs = ceil(2^32 / Cs): exact while k * Cs < 2^32 (cl_fits keeps k below 2^16 + 2^12 and Cs up to 2^15).
struct ClDiv { unsigned long long inv_wo; unsigned inv_kw, inv_cs; };

// What the kernel's index arithmetic takes: the packed filter matrix of a row tile stays below 2^31 bytes, and the products above hold.
CB_HD bool cl_fits(int Cs, int taps) { return Cs <= 32768 && (long long)Cs * taps <= 65536; }

inline ClDiv cl_div(int Wo, int Ho, int kw, int Cs = 4)
{
    ClDiv d;
    d.inv_wo = Wo < 4096 && Ho <= (1 << 22) ? ((1ull << 42) + (unsigned)Wo - 1ull) / (unsigned)Wo : 0ull;
    d.inv_kw = (65536u + (unsigned)kw - 1u) / (unsigned)kw;
    d.inv_cs = (unsigned)(((1ull << 32) + (unsigned)Cs - 1ull) / (unsigned)Cs);
    return d;
}

// tap of value k of a filter (Cs > 1)
CB_HD unsigned cl_tap(const ClDiv& d, unsigned k) { return (unsigned)(((unsigned long long)k * d.inv_cs) >> 32); }

// The piece that lies dt taps and cl < Cs channels behind value kb of a filter: its tap, and its channel less cl (modulo 2^32).  kb is the
// same for a whole workgroup, so its division is the scalar unit's.
CB_HD void cl_piece(const ClDiv& d, unsigned Cs, unsigned kb, unsigned dt, unsigned cl, unsigned& tap, unsigned& coff)
{
    const unsigned tb = cl_tap(d, kb), s = kb - tb * Cs;
    const bool next = s + cl >= Cs;
    tap = tb + dt + (next ? 1u : 0u);
    coff = s - (next ? Cs : 0u);
}

CB_HD int cl_row(const ClDiv& d, int q, int Wo) { return d.inv_wo ? (int)(((unsigned long long)(unsigned)q * d.inv_wo) >> 42) : q / Wo; }

// The kernel's instance: rows of its widest tile for O output channels, and 129 for bfloat16 layers whose maps (Po outputs) hold four
// 128 x 128 tiles per compute unit: the one with that tile.  (It needs registers that the narrow tiles then lack: 128 -> 96, 3x3, 92x164,
// 612 listed pixels 17.5 -> 19.1 us a frame with it.)
inline int cl_shape(int O, int Po, bool f32)
{
    return O <= 16 ? 16 : O <= 32 ? 32 : O <= 64 ? 64 : !f32 && (Po + 127LL) / 128 * ((O + 127LL) / 128) >= 1024 ? 129 : 128;
}

// Tiles (rows x columns) of instance `shape`: number 0 is 16 x 16 with the four wavefronts sharing K, the others follow.
//   16: 16 x 64, 16 x 128    32: 32 x 32, 32 x 64, 32 x 128    64: 64 x 16, 64 x 32, 64 x 64    128: 64 x 16, 64 x 32, 128 x 32, 128 x 64
//   129: these and 128 x 128
CB_HD constexpr int cl_tiles(int shape) { return shape == 16 ? 3 : shape == 128 ? 5 : shape == 129 ? 6 : 4; }

// Which tile finishes a frame first, in ns.  The kernel takes as long as the compute unit with the most tiles, and n tiles
// on it take about max(latency of one, n * its share of a busy unit) beyond the launch; both grow with the k-groups of the
// layer.  Fitted to every tile forced in turn (K = 288 to 12 544, 24 to 307 200 listed pixels, O = 8 to 512, both types):
// the choice is within a few percent of the best tile.
// N up to which the costs of O output channels fit 32 bits, whatever the filter (2 048 k-groups); with more listed pixels the tiles compare as they do with so many
CB_HD int cl_cost_pixels(int N, int O)
{
    const int most = (1 << 30) >> (32 - __builtin_clz((unsigned)O));
    return N < most ? N : most;
}
template <int BM, int BN> CB_HD unsigned cl_cost(int N, int O, unsigned nkg, unsigned l0, unsigned l1, unsigned c0, unsigned c1)
{
    const unsigned tiles = (((unsigned)N + BN - 1u) / BN) * (((unsigned)O + BM - 1u) / BM);
    const unsigned lat = l0 + l1 * nkg, busy = (tiles + 255u) / 256u * (c0 + c1 * nkg);
    return busy > lat ? busy : lat;
}

// run(number of the tile, a compile-time constant) for N listed pixels, O output channels, Cs channels of a pixel in the shadow,
// taps of the filter, R values of a filter.  (A function that returns the number instead cost the kernel registers: 128 -> 128
// bfloat16 at 1080p 453 -> 458 us.)
template <bool F32, int SHAPE, typename FN> CB_HD void cl_tile(int N, int O, int Cs, int taps, int R, FN&& run)
{
    N = cl_cost_pixels(N, O);
    // (literal arguments, not a table: a table would be fetched from memory ahead of everything else)
    const unsigned nkg = ((unsigned)(Cs * taps) + 31u) / 32u;
#define CB_COST(bm, bn, a0, a1, a2, a3, b0, b1, b2, b3) \
    (F32 ? cl_cost<bm, bn>(N, O, nkg, a0, a1, a2, a3) : cl_cost<bm, bn>(N, O, nkg, b0, b1, b2, b3))
    // 16 x 16, the four wavefronts sharing K: four times the tiles of the others where few pixels are listed, a quarter of
    // the serial chain (256 -> 8, 7x7, 3 322 pixels: 104 -> 43 us; 64 -> 9, 3x3: 8.7 -> 6.5 us)
    // (filters beyond one XCD's 4 MB of L2 come in more slowly than its four wavefronts ask for them: 512 -> 512, 324 pixels
    // 42 us, 33 us with 64 x 16)
    const bool far = F32 && (unsigned long long)O * (unsigned)R > 700000ull;
    const unsigned k = CB_COST(16, 16, 100, 94, 1260, (far ? 80 : 49), 200, 30, 870, 16);
    if constexpr (SHAPE == 16) {
        const unsigned a = CB_COST(16, 64, 1600, 330, 1100, 222, 200, 110, 1000, 60), b = CB_COST(16, 128, 2600, 700, 1300, 440, 300, 200, 1300, 110);
        if (k <= a && k <= b) run(std::integral_constant<int, 0>());
        else if (a <= b) run(std::integral_constant<int, 1>());
        else run(std::integral_constant<int, 2>());
    } else if constexpr (SHAPE == 32) {
        const unsigned a = CB_COST(32, 32, 200, 230, 1250, 155, 200, 70, 850, 50), b = CB_COST(32, 64, 600, 390, 1200, 290, 400, 120, 800, 85),
                       c = CB_COST(32, 128, 1000, 800, 1500, 550, 900, 220, 900, 130);
        if (k <= a && k <= b && k <= c) run(std::integral_constant<int, 0>());
        else if (a <= b && a <= c) run(std::integral_constant<int, 1>());
        else if (b <= c) run(std::integral_constant<int, 2>());
        else run(std::integral_constant<int, 3>());
    } else if constexpr (SHAPE == 64) {
        const unsigned a = CB_COST(64, 16, 0, 176, 1250, 120, 100, 58, 650, 41), b = CB_COST(64, 32, 1600, 310, 1400, 200, 400, 83, 1100, 48),
                       c = CB_COST(64, 64, 1300, 530, 800, 395, 1000, 148, 800, 100);
        if (k <= a && k <= b && k <= c) run(std::integral_constant<int, 0>());
        else if (a <= b && a <= c) run(std::integral_constant<int, 1>());
        else if (b <= c) run(std::integral_constant<int, 2>());
        else run(std::integral_constant<int, 3>());
    } else {
        // (128 x 32 in bfloat16: 95 a group instead of 100 takes it from 144 groups on where two rounds of 64 x 32 are faster,
        // 512 -> 512, 3x3, 1 425 pixels 22.0 against 21.2 us)
        const unsigned a = CB_COST(64, 16, 0, 176, 1250, 120, 100, 58, 650, 41), b = CB_COST(64, 32, 1000, 300, 1400, 203, 400, 80, 1100, 47),
                       c = CB_COST(128, 32, 1800, 380, 1000, 320, 1500, 100, 100, 96), d = CB_COST(128, 64, 900, 745, 2900, 510, 2000, 190, 1000, 140),
                       ab = a < b ? a : b, cd = c < d ? c : d;
        // 128 x 128 halves what a column costs in filter fragments and gathers; from two tiles per compute unit on, so that they
        // have others to run beside.  us, 128 x 64 / 128 x 128: 64 -> 128, 1x1, 101 376 pixels 33 / 20; 128 -> 256, 1x1, 41 216 in blocks 29 / 18;
        // 64 -> 96, 3x3, 122 187 56 / 34; 128 -> 512, 3x3, 233 661 420 / 358; 64 -> 256, 7x7, 151 306 294 / 254; 64 -> 128, 3x3, 1080p, 5 %
        // changed 64 / 51.  Where sparse outputs of 60 - 150 MB bound both by their writes a frame takes up to 1.6 % more (128 -> 128, 3x3, 1080p,
        // 10 %: 452.5 / 457.5); a test for that here cost the other layers as much.  (float32 has no registers for it.  The cost is compared with that of 128 x 64 alone: those of the narrower
        // tiles miss what many listed pixels pay for their stores, 1x1 above all.)
        if (SHAPE == 129 && (((unsigned)N + 127u) / 128u) * (((unsigned)O + 127u) / 128u) >= 512u && cl_cost<128, 128>(N, O, nkg, 1500, 420, 1000, 250) <= d)
            run(std::integral_constant<int, SHAPE == 129 ? 5 : 4>());
        else if (k <= ab && k <= cd) run(std::integral_constant<int, 0>());
        else if (ab <= cd) { if (a <= b) run(std::integral_constant<int, 1>()); else run(std::integral_constant<int, 2>()); }
        else if (c <= d) run(std::integral_constant<int, 3>());
        else run(std::integral_constant<int, 4>());
    }
#undef CB_COST
}

// Size of a packed filter matrix of nkg k-groups (bfloat16 64 bytes a group and row, float32 three such terms), and from which on its rows
// are divided among the XCDs
CB_HD unsigned cl_filter_kb(int O, unsigned nkg, bool f32) { return ((unsigned)O * nkg >> 4) * (f32 ? 3u : 1u); }
constexpr unsigned CL_FAR_KB = 2048;
CB_HD unsigned cl_pixel_kb(unsigned N, unsigned Cs, unsigned esz) { return N * (Cs * esz / 16u) >> 6; }

// Logarithm of the groups of XCDs among which the row tiles (MT) are divided; the column tiles are divided among the XCDs of a group.
// Each XCD brings its rows of the filter matrix (filter_kb in all) and the pixels of its columns (pixel_kb, about) into its own L2: 2^l groups
// move filter_kb * 8 / 2^l + pixel_kb * 2^l.  Filters are fetched several groups ahead, pixels one stage, so that a miss of a pixel
// costs more: they count fourfold (counted once: ten-layer trunk of 3 x 3 filters at 368x656, float32, 282 us, fourfold 279; 512 -> 512 at 46x82, bfloat16, 10 % 41.9 / 41.5).
// Filters of up to 2 MB stay in every L2 beside the pixels and gain nothing.  Frames, us, undivided / divided: 512 -> 512, 3x3, 46x82, 2 % changed
// 45.3 / 42.2, bfloat16 35.7 / 33.9, 30 % 46.5 / 46.8; 256 -> 512 there 28.9 / 26.9; 256 -> 256, 3x3, 92x164 31.3 / 30.0; 64 -> 256, 7x7, 120x160
// 53.5 / 52.2; below the line 128 -> 256, 3x3, 184x328 (1.8 MB) 39.1 / 39.7.
// Groups among which the tiles (NT column tiles, an item each or `parts`) do not come out even keep some XCDs waiting for others: at most an eighth
// more items on one than undivided, or one for each of its 32 compute units.  Without that limit, frames, us, undivided / divided: 128 -> 330, 5x5, 60x80, 30 % 57.4 / 68.2,
// every output 79.1 / 90.1, bfloat16 35.2 / 40.8; 512 -> 520, 3x3, 46x82, 30 % 89.5 / 96.7.
CB_HD unsigned cl_xcd_tiles(unsigned MT, unsigned NT, unsigned l) { return ((NT + (8u >> l) - 1u) >> (3u - l)) * ((MT + (1u << l) - 1u) >> l); }
CB_HD unsigned cl_xcd_rows(unsigned MT, unsigned NT, unsigned parts, unsigned filter_kb, unsigned pixel_kb)
{
    unsigned l = filter_kb / 16u > pixel_kb ? 3u : filter_kb / 4u > pixel_kb ? 2u : filter_kb > pixel_kb ? 1u : 0u;
    const unsigned most = cl_xcd_tiles(MT, NT, 0u) * 9u / 8u;
    // (a loop: every workgroup fetches this code before its first load)
#ifdef __HIPCC__
#pragma unroll 1
#endif
    for (; l > 0u; --l) {
        const unsigned tiles = cl_xcd_tiles(MT, NT, l);
        if ((1u << l) <= MT && (tiles <= most || tiles * parts <= 32u)) break;
    }
    return l;
}

// Whether the K of a layer with such filters is divided, and into how many parts: 0, or parts + 16 * (128 x 64 instead of 128 x 32 tiles).
// A few hundred tiles leave compute units idle in the last of one or two rounds, and tiles narrow enough to fill them fetch filters and pixels several times as
// often; wide tiles in parts do neither.  The price is CL_SPLIT_NS: sums written through to memory, counted, read back.  Costs as in cl_tile.
// Frames, us, whole / divided: float32 512 -> 512, 3x3, 46x82, 2 and 10 % changed 45.5 / 35.8, 30 % 74.7 / 60.3, every output 113.5 / 109.2; 64 -> 256, 7x7, 30x40
// 30.3 / 24.2, but 120x160, 10 % 55.1 / 56.1; 128 -> 128, 9x9, 60x80 44.8 / 37.8; 256 -> 128 there 77.5 / 56.7; bfloat16 256 -> 256, 7x7, 60x80, 20 % 55.0 / 44.8.  Shorter filters
// are not considered, for which the choice alone took 0.4 us: 256 -> 256, 3x3, 92x164 (72 groups) 29.7 / 30.6; bfloat16 512 -> 512, 3x3, 46x82 (144) 42.3 / 43.0.
// float32: K is only divided where that rounds the sums no worse than the whole tile.  Relative errors of sums over a K of 4 608 against float64: one
// chain of products 1.06e-6, two (the small terms in one of their own: up to four tiles a wavefront) 4.1e-7, groups of six products added at once (128 x 64) 2.5e-7, two in each of four wavefronts
// that share K 1.9e-7; in p parts they fall with the square root of p.  The numbers of parts are those for a 128 x 64 tile of one chain, which it was when they were fitted: 2 of its parts are as exact as any
// whole tile now, and the costs of more layers in so few are not measured.
constexpr unsigned CL_SPLIT_NS = 8500, CL_SPLIT_MAX = 8;     // (tiles: at most 256)
// the fewest parts of a 128 x 64 tile as one chain (or of 128 x 32, two) that are as exact as a whole tile: 0: 64 x 16 and 64 x 32, 1: 16 x 16, 2: 128 x 32 and 128 x 64
CB_HD unsigned cl_least_parts(int whole, bool two) { return whole == 2 ? 2u : whole == 0 ? (two ? 2u : 7u) : two ? 5u : CL_SPLIT_MAX + 1u; }
CB_HD bool cl_split_pays(unsigned nkg, bool f32) { return nkg >= (f32 ? 96u : 256u); }
template <bool F32> CB_HD unsigned cl_split(int N, int O, unsigned nkg, unsigned ws_bytes)
{
    if (N > cl_cost_pixels(N, O)) return 0;       // (far more tiles than parts are considered for)
#define CB_COST(bm, bn, n, a0, a1, a2, a3, b0, b1, b2, b3) \
    (F32 ? cl_cost<bm, bn>(n, O, nkg, a0, a1, a2, a3) : cl_cost<bm, bn>(n, O, nkg, b0, b1, b2, b3))
    const unsigned a = CB_COST(64, 16, N, 0, 176, 1250, 120, 100, 58, 650, 41), b = CB_COST(64, 32, N, 1000, 300, 1400, 203, 400, 80, 1100, 47),
                   c = CB_COST(128, 32, N, 1800, 380, 1000, 320, 1500, 100, 100, 96), d = CB_COST(128, 64, N, 900, 745, 2900, 510, 2000, 190, 1000, 140),
                   k = CB_COST(16, 16, N, 100, 94, 1260, (O * (unsigned long long)nkg > 700000ull / 32u ? 80 : 49), 200, 30, 870, 16);
#undef CB_COST
    unsigned best = a < b ? a : b, choice = 0;
    best = best < c ? best : c;
    best = best < d ? best : d;
    best = best < k ? best : k;
    if (best < CL_SPLIT_NS) return 0;
    const int whole = best == k ? 1 : best == a || best == b ? 0 : 2;        // (of equal ones the most exact)
    // as many parts as make one or two items per compute unit
    // (of the tiles of the busiest XCD, with as many groups as the row tiles come out even in: the rule of cl_xcd_rows here took 0.5 us of a launch)
    const unsigned rows = ((unsigned)O + 127u) / 128u, even = rows & 1u ? 0u : rows & 2u ? 1u : rows & 4u ? 2u : 3u;
    // (an XCD's compute units take what falls to that XCD: 512 -> 260, 3x3, 46x82, 30 %, 432 items of which one XCD had 80, not 54, whole 58.7, divided 64.5)
    auto consider = [&](unsigned cols, unsigned flag, unsigned bytes, unsigned l0, unsigned l1, unsigned c0, unsigned c1) {
        const unsigned tiles = cols * rows;
        if (tiles > 256u) return;
        const unsigned on_one = cl_xcd_tiles(rows, cols, even);
        const unsigned one = 256u / tiles, two = 512u / tiles;
        for (unsigned r = 0; r < 2; ++r) {
            unsigned p = r ? two : one;
            p = p > CL_SPLIT_MAX ? CL_SPLIT_MAX : p;
            const unsigned g = (nkg + p - 1u) / p;
            if (p < (F32 ? cl_least_parts(whole, !flag) : 2u) || g < 8u || tiles * p * bytes > ws_bytes) continue;
            const unsigned lat = l0 + l1 * g, busy = (on_one * p + 31u) / 32u * (c0 + c1 * g), v = (busy > lat ? busy : lat) + CL_SPLIT_NS;
            if (v < best) { best = v; choice = p | flag; }
        }
    };
    consider(((unsigned)N + 31u) / 32u, 0u, 16384u, F32 ? 1800u : 1500u, F32 ? 380u : 100u, F32 ? 1000u : 100u, F32 ? 320u : 96u);
    consider(((unsigned)N + 63u) / 64u, 16u, 32768u, F32 ? 900u : 2000u, F32 ? 745u : 190u, F32 ? 2900u : 1000u, F32 ? 510u : 140u);
    return choice;
}

}  // namespace cb
