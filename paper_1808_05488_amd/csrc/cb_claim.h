// Who does what in a launch in which workgroups that extract wait for workgroups that detect: plain logic, usable from host code and
// kernels alike.
//
// A workgroup must not wait for one that has not begun: the places that one needs may be taken by workgroups that wait, of this launch (few compute
// units: a partitioned device, a masked queue) or of others (streams, processes), and nobody would ever leave.  So a block of detection
// belongs to whoever claims it first: its own workgroup, as it begins, or an extracting one that has waited for a while and finds it unclaimed.  What
// is claimed is being worked on by a workgroup that runs and waits for nothing.  Only when every block is claimed does an extracting workgroup
// wait without a limit.  Nothing is assumed about the size of the chip, the order of dispatch or what else runs.
//
// A claim is the frame's tag, exchanged into the block's word: whoever finds another value there has the block, and nothing needs clearing.  The
// frame count, from which a workgroup knows the tag, must not advance before the last workgroup has begun: `done` counts the extracting workgroups
// that are through and, in units of CLAIM_TAKEN, the blocks taken from workgroups that have not come by yet; whoever completes it ends the frame.
#pragma once

#ifndef CB_HD
#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define CB_HD __host__ __device__ __forceinline__
#else
#define CB_HD inline
#endif
#endif

namespace cb {

// (up to 512 workgroups extract.  2^22 blocks taken at once would overflow; a launch has at most 2^19.)
constexpr int CLAIM_TAKEN = 1024;

// The word of block b of n.  Blocks that begin together have theirs on different cache lines: atomics of one line queue up at memory.
CB_HD constexpr unsigned claim_words(unsigned n) { return 32u * (((n >> 5) + 32u) & ~31u); }
CB_HD constexpr unsigned claim_index(unsigned b, unsigned n) { return (b & 31u) * (((n >> 5) + 32u) & ~31u) + (b >> 5); }

// MEM: exchange(word, value) and add(word, value) return what was there; both are atomic, and add is complete when it returns.
// Claims a block for its own workgroup, or for another (taking): what its word held.  The tag: somebody has it.
template <typename MEM, typename W, typename D> CB_HD unsigned claim_block(MEM&& mem, W* claim, unsigned tag, D* done, bool taking)
{
    if (taking) mem.add(done, CLAIM_TAKEN);
    return mem.exchange(claim, tag);
}
// ... if somebody has it: true if the frame is over
template <typename MEM, typename D> CB_HD bool claim_lost(MEM&& mem, D* done, int extracting) { return mem.add(done, -CLAIM_TAKEN) == extracting + CLAIM_TAKEN; }
// an extracting workgroup is through: true if the frame is over
CB_HD constexpr bool extraction_last(int before, int extracting) { return before == extracting - 1; }
template <typename MEM, typename D> CB_HD bool extraction_done(MEM&& mem, D* done, int extracting) { return extraction_last(mem.add(done, 1), extracting); }

// Row of word `it` of a map of w words a row, with inv = map_row_inv(w): exact while it * w < 2^31.  (Maps that are extracted in the launch of detection have at most 2^17
// words, and rows of at most 2^11.)
inline unsigned map_row_inv(unsigned w) { return (0x80000000u + w - 1u) / w; }
CB_HD unsigned map_row(unsigned it, unsigned inv) { return (unsigned)(((unsigned long long)it * inv) >> 31); }

// The number of an extracting workgroup, in the order in which they begin: it waits, without a limit, for what those with lower numbers publish, and each publishes
// before it waits for any of them.
template <typename MEM, typename D> CB_HD int extraction_number(MEM&& mem, D* begun) { return mem.add(begun, 1); }

// One workgroup, all of its threads together.  extracts: its role, by number; detect(): claims its block of detection and does it; unclaimed(): some block
// that nobody has claimed, -1: none; take(block): claims it and does it; await(limited): until what this workgroup extracts from is there, or (limited) until
// its patience runs out: false.
template <typename DETECT, typename AWAIT, typename UNCLAIMED, typename TAKE, typename EXTRACT>
CB_HD void detect_or_extract(bool extracts, DETECT&& detect, AWAIT&& await, UNCLAIMED&& unclaimed, TAKE&& take, EXTRACT&& extract)
{
    if (!extracts) {
        detect();
        return;
    }
    if (!await(true)) {
        for (int b = unclaimed(); b >= 0; b = unclaimed()) take(b);
        await(false);
    }
    extract();
}

}  // namespace cb
