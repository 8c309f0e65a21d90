// Change-map dilation by the filter footprint (Sec. III-A Eq. 4) and change-index
// extraction (Sec. III-A, "Change Indexes Extraction"), on bit-packed maps.
//
// The paper sets the k x k neighbourhood of every changed pixel (scatter form)
// and compacts with a library stream-compaction call.  Here the map is held as
// 64-pixel words: one thread produces one word of the dilated map from at most
// three input words per filter row (shifts and ORs), the words' popcounts are
// scanned (wavefront moves + LDS), and set bits are expanded into the ordered
// index list a word at a time by a whole wavefront (one-workgroup kernel: sparse words by their lane).  No atomics on
// the ordering path, so the list is strictly ascending by construction.
//
//   dilate_kernel : word (yo, wo) of the dilated map + per-block popcount
//   compact_kernel: block prefix over the popcounts, in-block scan, index write, N
//   dilate_compact_small_kernel: both in one workgroup, for maps of up to 1024 words
//                   (launch latency, not work, is what these steps cost there)
//   dilate_compact_kernel: both in one launch of many workgroups (single-pass scan), for
//                   maps of up to 262 144 words; the two-kernel form remains for larger ones
#include "cb_extract.h"

namespace cb {

namespace {

__global__ __launch_bounds__(256) void dilate_kernel(Geom g, const uint64_t* __restrict__ in_bits,
                                                     long pitch, int full, uint64_t* __restrict__ mt_bits,
                                                     int* __restrict__ blk_cnt, int* __restrict__ ctl, int own_map,
                                                     int clear_words)
{
    __shared__ int wsum[4];
    __shared__ uint64_t s_map[MAP_STAGE];
    const int items = g.Ho * g.WWo;
    const int it = blockIdx.x * 256 + threadIdx.x;
    const int par = frame_parity(ctl, own_map);
    uint64_t word = 0;
    if (!full) word = dilated_block_word<256, MAP_STAGE>(g, in_bits, pitch, (int)blockIdx.x * 256, items, own_map, par, s_map);
    if (it < items) {
        if (full) word = full_word(g, it);
        mt_bits[it] = word;
    }
    if (own_map) clear_other_map(const_cast<uint64_t*>(in_bits), ctl, par, clear_words, it, (int)gridDim.x * 256);
    int s = wave_sum(__popcll(word));
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        blk_cnt[blockIdx.x] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    }
}

__global__ __launch_bounds__(256) void compact_kernel(Geom g, const uint64_t* __restrict__ mt_bits,
                                                      const int* __restrict__ blk_cnt,
                                                      int32_t* __restrict__ idx, int* __restrict__ ctl, int own_map)
{
    __shared__ int red[4];
    __shared__ int wtot[4];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int items = g.Ho * g.WWo;

    // exclusive prefix of the counts of all earlier blocks
    int part = 0;
    for (int b = tid; b < (int)blockIdx.x; b += 256) part += blk_cnt[b];
    part = wave_sum(part);
    if (lane == 0) red[wv] = part;

    const int it = blockIdx.x * 256 + tid;
    uint64_t word = 0;
    int pixbase = 0;
    if (it < items) {
        word = mt_bits[it];
        const int yo = it / g.WWo, wo = it - yo * g.WWo;
        pixbase = yo * g.Wo + 64 * wo;
    }
    const int cnt = __popcll(word);
    const int inc = wave_inclusive_scan(cnt);                  // inclusive scan inside the wavefront
    if (lane == 63) wtot[wv] = inc;
    __syncthreads();
    int off = red[0] + red[1] + red[2] + red[3];
    for (int q = 0; q < wv; ++q) off += wtot[q];
    off += inc - cnt;                       // exclusive offset of this thread's word

    if (blockIdx.x == gridDim.x - 1 && tid == 255) {
        ctl[CTL_COUNT] = off + cnt;
        if (own_map) ctl[CTL_FRAME] = ctl[CTL_FRAME] + 1;     // (the dilation kernel, which read it, is complete)
    }

    expand_words<false>(word, off, pixbase, idx, lane);
}

// Dilation, scan and index write in ONE launch for maps of up to ONE_PASS_MAX_BLOCKS x 256 words.
// The scan over workgroups is a single-pass one: every workgroup publishes the popcount of its 256
// words and then adds up what its predecessors published, so nobody waits for a chain of prefixes.
// Progress: a workgroup publishes its own count before it waits for anybody, and it only waits for
// workgroups with lower numbers, which were dispatched no later than itself and publish before they
// wait in turn; on an idle GPU the whole grid (at most 1024 workgroups of 256 threads, 93 registers and
// 16.4 KB of LDS: five per compute unit, 1 280 on the chip) is resident at once anyway.  Correctness does not rest on either: the
// wait is bounded (spin_limit polls per predecessor), and a thread whose wait runs out -- other
// streams or processes may hold the compute units the predecessor is waiting for -- recomputes that
// predecessor's count itself from the input map (recount_block), which needs nobody else.  The list
// and N are therefore the same whatever the scheduling; CTL_RECOUNTS only counts how often that
// happened.  Published counts carry the launch's epoch in their upper half, so the slots never need
// clearing; the last workgroup to finish stores the epoch in device memory for the next launch
// (nothing launch-specific comes from the host, so a captured launch can be replayed).
constexpr int ONE_PASS_MAX_BLOCKS = 1024;

// Number of set bits in workgroup b's 256 words of the dilated map, from the input map alone.
// (inlined: a call would give the kernel a stack, and with it a slower launch, for a path that an idle GPU never takes)
__device__ __forceinline__ int recount_block(const Geom& g, const uint64_t* __restrict__ in_bits, long pitch, int full,
                                          int b, int own_map, int par)
{
    const int items = g.Ho * g.WWo;
    const int hi = b * 256 + 256 < items ? b * 256 + 256 : items;
    int total = 0;
    for (int it = b * 256; it < hi; ++it) {
        const int yo = it / g.WWo, wo = it - yo * g.WWo;
        if (full) total += __popcll(full_word(g, it));
        else total += __popcll(dilated_word(g, in_bits, pitch, yo, wo, own_map, par));
    }
    return total;
}

__global__ __launch_bounds__(256) void dilate_compact_kernel(Geom g, const uint64_t* __restrict__ in_bits,
                                                             long pitch,
                                                             int full, uint64_t* __restrict__ mt_bits,
                                                             int32_t* __restrict__ idx, int* __restrict__ ctl,
                                                             unsigned long long* __restrict__ look, int own_map,
                                                             int clear_words, int spin_limit)
{
    // (needed only after the map words have been requested: both candidates come with one load)
    const int par = frame_parity(ctl, own_map);
    __shared__ unsigned s_small[ONE_PASS_SMALL];
    __shared__ uint64_t s_map[MAP_STAGE];
    const int tid = threadIdx.x;
    const int items = g.Ho * g.WWo;
    const int nblk = (int)gridDim.x;
    // written by the previous launch's last workgroup; the load is in flight during the dilation
    unsigned epoch_ld = tid == 0 ? (unsigned)ctl[CTL_EPOCH] : 0u;
    const int bid = (int)blockIdx.x;

    const int it = bid * 256 + tid;
    uint64_t word = 0;
    int pixbase = 0;
    if (!full) word = dilated_block_word<256, MAP_STAGE>(g, in_bits, pitch, bid * 256, items, own_map, par, s_map);
    if (it < items) {
        const int yo = it / g.WWo, wo = it - yo * g.WWo;
        if (full) word = full_word(g, it);
        mt_bits[it] = word;
        pixbase = yo * g.Wo + 64 * wo;
    }
    // housekeeping for the next frame: the other input map starts out empty
    if (own_map) clear_other_map(const_cast<uint64_t*>(in_bits), ctl, par, clear_words, bid * 256 + tid, nblk * 256);
    one_pass_tail(word, pixbase, epoch_ld, idx, ctl, look, own_map, bid, nblk, spin_limit, s_small,
                  [&](int b) { return recount_block(g, in_bits, pitch, full, b, own_map, par); });
}

// Small maps: dilation, scan and index write in ONE workgroup of 1024 threads, so
// that the whole change-index extraction costs a single launch.  The workgroup walks
// the words in rounds of 1024, carrying the running count.
__global__ __launch_bounds__(1024) void dilate_compact_small_kernel(Geom g, const uint64_t* __restrict__ in_bits,
                                                                    long pitch, int full,
                                                                    uint64_t* __restrict__ mt_bits,
                                                                    int32_t* __restrict__ idx, int* __restrict__ ctl,
                                                                    int own_map, int clear_words)
{
    const int par = frame_parity(ctl, own_map);
    __shared__ int wtot[16];
    __shared__ int carry;
    __shared__ uint64_t s_map[MAP_STAGE_SMALL];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int items = g.Ho * g.WWo;
    if (tid == 0) carry = 0;
    for (int r0 = 0; r0 < items; r0 += 1024) {
        const int it = r0 + tid;
        uint64_t word = 0;
        int pixbase = 0;
        if (!full) word = dilated_block_word<1024, MAP_STAGE_SMALL>(g, in_bits, pitch, r0, items, own_map, par, s_map);
        if (it < items) {
            const int yo = it / g.WWo, wo = it - yo * g.WWo;
            if (full) word = full_word(g, it);
            mt_bits[it] = word;
            pixbase = yo * g.Wo + 64 * wo;
        }
        const int cnt = __popcll(word);
        const int inc = wave_inclusive_scan(cnt);                  // inclusive scan inside the wavefront
        __syncthreads();                 // previous round's wtot / carry have been consumed
        if (lane == 63) wtot[wv] = inc;
        __syncthreads();
        int off = carry;
        for (int q = 0; q < wv; ++q) off += wtot[q];
        off += inc - cnt;
        int round_total = 0;
        for (int q = 0; q < 16; ++q) round_total += wtot[q];
        // mostly full words (a full update): one word at a time after all, 64 stores to 64 lines per
        // instruction cost more there (15 088 listed pixels of 92x164: 10.7 -> 7.5 us)
        if (__builtin_amdgcn_readlane(inc, 63) >= 2048) expand_words<false>(word, off, pixbase, idx, lane);
        else expand_words<true>(word, off, pixbase, idx, lane);
        __syncthreads();                 // everyone has read carry
        if (tid == 0) carry += round_total;
    }
    if (own_map) clear_other_map(const_cast<uint64_t*>(in_bits), ctl, par, clear_words, tid, 1024);
    __syncthreads();
    if (tid == 0) {
        ctl[CTL_COUNT] = carry;
        if (own_map) ctl[CTL_FRAME] = ctl[CTL_FRAME] + 1;    // (one workgroup: everybody is past its reads)
    }
}

__global__ __launch_bounds__(256) void expand_bits_kernel(const uint64_t* __restrict__ bits, long pitch,
                                                          int H, int W, uint8_t* __restrict__ bytes)
{
    const long n = (long)H * W;
    for (long q = (long)blockIdx.x * 256 + threadIdx.x; q < n; q += (long)gridDim.x * 256) {
        const int y = (int)(q / W), x = (int)(q - (long)y * W);
        bytes[q] = test_bit<false>(bits, (long)y * pitch + x, 0) ? 1 : 0;
    }
}

// The input map of the last processed frame of a layer that detects its own changes: of its two
// interleaved maps the one that the frame count on the device selected for that frame.
__global__ __launch_bounds__(256) void expand_own_map_kernel(const uint64_t* __restrict__ bits,
                                                             const int* __restrict__ ctl, long pitch, int H, int W,
                                                             uint8_t* __restrict__ bytes)
{
    const int par = (ctl[CTL_FRAME] - 1) & 1;
    const long n = (long)H * W;
    for (long q = (long)blockIdx.x * 256 + threadIdx.x; q < n; q += (long)gridDim.x * 256) {
        const int y = (int)(q / W), x = (int)(q - (long)y * W);
        bytes[q] = test_bit<true>(bits, (long)y * pitch + x, par) ? 1 : 0;
    }
}

__global__ __launch_bounds__(256) void fill32_kernel(uint32_t* __restrict__ p, size_t n, uint32_t v)
{
    for (size_t q = (size_t)blockIdx.x * 256 + threadIdx.x; q < n; q += (size_t)gridDim.x * 256) p[q] = v;
}

// Pooled change map: bit (yp, xp) = OR over the w x w window of the producer's
// dilated map (row-padded words in, row-padded words out).
__global__ __launch_bounds__(256) void pool_mask_kernel(int Ho, int Wo, int WWo, int w, int Hp, int Wp, int WWp,
                                                        const uint64_t* __restrict__ mt_bits,
                                                        uint64_t* __restrict__ pm_bits)
{
    const int items = Hp * WWp;
    const int it = blockIdx.x * 256 + threadIdx.x;
    if (it >= items) return;
    const int yp = it / WWp, wp = it - yp * WWp;
    if (w == 2) {
        pm_bits[it] = pooled_word(mt_bits, Ho, WWo, yp, wp);
        return;
    }
    uint64_t word = 0;
    for (int b = 0; b < 64; ++b) {
        const int xp = 64 * wp + b;
        if (xp >= Wp) break;
        bool any = false;
        for (int dy = 0; dy < w; ++dy)
            for (int dx = 0; dx < w; ++dx) {
                const int y = yp * w + dy, x = xp * w + dx;
                if (y < Ho && x < Wo && test_bit<false>(mt_bits, ((long)y * WWo << 6) + x, 0)) any = true;
            }
        word |= (uint64_t)any << b;
    }
    pm_bits[it] = word;
}

}  // namespace

int dilate_num_blocks(const Geom& g) { return (g.Ho * g.WWo + 255) / 256; }

// one round of the one-workgroup kernel; beyond that its serial rounds cost more than a second launch
bool compact_single_launch(const Geom& g) { return g.Ho * g.WWo <= 1024; }

hipError_t launch_dilate_compact_small(const Geom& g, const uint64_t* in_bits, long in_pitch_bits,
                                       int full, uint64_t* mt_bits, int32_t* idx, int* ctl, int own_map,
                                       int clear_words, hipStream_t st, Tm tm)
{
    CB_LAUNCH(dilate_compact_small_kernel, dim3(1), dim3(1024), st, tm, g, in_bits, in_pitch_bits, full,
              mt_bits, idx, ctl, own_map, clear_words);
    return hipGetLastError();
}

// (the input map of such a consumer has rows of whole words)
bool extract_fits(const Geom& g)
{
    const long rows = (long)((255 + g.WWo - 1) / g.WWo) * g.s + g.kh, n = rows * ((g.W + 63) / 64) + 3;
    return n <= MAP_STAGE && dilate_num_blocks(g) <= 256;
}

bool compact_one_pass(const Geom& g) { return dilate_num_blocks(g) <= ONE_PASS_MAX_BLOCKS; }
size_t compact_one_pass_bytes(const Geom& g) { return compact_one_pass(g) ? (size_t)dilate_num_blocks(g) * 8 : 0; }

hipError_t launch_dilate_compact(const Geom& g, const uint64_t* in_bits, long in_pitch_bits, int full,
                                 uint64_t* mt_bits, int32_t* idx, int* ctl, uint64_t* look, int own_map,
                                 int clear_words, int spin_limit, hipStream_t st, Tm tm)
{
    CB_LAUNCH(dilate_compact_kernel, dim3(dilate_num_blocks(g)), dim3(256), st, tm, g, in_bits,
              in_pitch_bits, full, mt_bits, idx, ctl, reinterpret_cast<unsigned long long*>(look), own_map, clear_words,
              spin_limit);
    return hipGetLastError();
}

hipError_t launch_dilate(const Geom& g, const uint64_t* in_bits, long in_pitch_bits, int full,
                         uint64_t* mt_bits, int* blk_cnt, int* ctl, int own_map, int clear_words, hipStream_t st, Tm tm)
{
    CB_LAUNCH(dilate_kernel, dim3(dilate_num_blocks(g)), dim3(256), st, tm, g, in_bits, in_pitch_bits,
              full, mt_bits, blk_cnt, ctl, own_map, clear_words);
    return hipGetLastError();
}

hipError_t launch_compact(const Geom& g, const uint64_t* mt_bits, const int* blk_cnt, int32_t* idx,
                          int* ctl, int own_map, hipStream_t st, Tm tm)
{
    CB_LAUNCH(compact_kernel, dim3(dilate_num_blocks(g)), dim3(256), st, tm, g, mt_bits, blk_cnt, idx, ctl, own_map);
    return hipGetLastError();
}

hipError_t launch_expand_own_map(const uint64_t* bits0, const int* ctl, long pitch_bits, int H, int W,
                                 uint8_t* bytes, hipStream_t st)
{
    long n = (long)H * W;
    unsigned grid = (unsigned)((n + 255) / 256);
    if (grid > 4096) grid = 4096;
    if (grid == 0) grid = 1;
    hipLaunchKernelGGL(expand_own_map_kernel, dim3(grid), dim3(256), 0, st, bits0, ctl, pitch_bits, H, W, bytes);
    return hipGetLastError();
}

hipError_t launch_expand_bits(const uint64_t* bits, long pitch_bits, int H, int W, uint8_t* bytes,
                              hipStream_t st)
{
    long n = (long)H * W;
    unsigned grid = (unsigned)((n + 255) / 256);
    if (grid > 4096) grid = 4096;
    if (grid == 0) grid = 1;
    hipLaunchKernelGGL(expand_bits_kernel, dim3(grid), dim3(256), 0, st, bits, pitch_bits, H, W, bytes);
    return hipGetLastError();
}

hipError_t launch_fill32(uint32_t* p, size_t n, uint32_t v, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    size_t grid = (n + 255) / 256;
    if (grid > 4096) grid = 4096;
    hipLaunchKernelGGL(fill32_kernel, dim3((unsigned)grid), dim3(256), 0, st, p, n, v);
    return hipGetLastError();
}

hipError_t launch_pool_mask(int Ho, int Wo, int WWo, int w, const uint64_t* mt_bits, uint64_t* pm_bits,
                            hipStream_t st)
{
    const int Hp = (Ho + w - 1) / w, Wp = (Wo + w - 1) / w, WWp = (Wp + 63) / 64;
    const int items = Hp * WWp;
    hipLaunchKernelGGL(pool_mask_kernel, dim3((items + 255) / 256), dim3(256), 0, st, Ho, Wo, WWo, w, Hp, Wp, WWp,
                       mt_bits, pm_bits);
    return hipGetLastError();
}

}  // namespace cb
