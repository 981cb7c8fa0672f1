// Internal: the arithmetic by which the host cuts a call into workgroups and launches and sizes the tables that the
// kernels look things up in.  Plain C++ without HIP, so that its limits can be tested without a GPU.
#ifndef FLASHOPTIM_LAUNCH_H
#define FLASHOPTIM_LAUNCH_H

#include <stdint.h>

namespace fo {

// A launch over a list maps workgroup b to (tensor, tile), or in a copy to (segment, piece), in two steps:
// coarse[b >> shift] is the table entry that holds workgroup (b >> shift) << shift, coarse[(b >> shift) + 1] the next such (behind
// the last one: the table's last entry), and entry_of searches between the two (usually they are the same).  Both tables
// are small (at most kCoarseMaxEntries coarse entries and one) and stay cache-resident, unlike a table with one entry per
// workgroup, whose entries every workgroup would fetch from HBM.
constexpr int64_t kCoarseMaxEntries = 16384;
// Coarse entries for `total` (>= 0) workgroups.
constexpr int64_t coarse_entries(int64_t total, uint32_t shift) { return total > 0 ? ((total - 1) >> shift) + 1 : 0; }
// The smallest shift with which they fit.
constexpr uint32_t coarse_shift(int64_t total) {
    uint32_t shift = 0;
    while (coarse_entries(total, shift) > kCoarseMaxEntries) ++shift;
    return shift;
}

// The entry that holds workgroup b: the last one of first .. last that begins at b or before it, begin(i) being entry i's first
// workgroup.  By bisection: beside a large tensor a coarse entry spans hundreds of workgroups, and as many entries of the table
// where a list has thousands of small tensors (one after the other -> by bisection: 30000 tensors of 1000 elements beside 100 M,
// compress 401.3 -> 383.7 us, decompress 405.0 -> 384.4; of 30 beside 300 M, 970 -> 840, 1079 -> 961, Lion 653 -> 620; 8000 tensors
// beside 16 GB, a checkpoint pack 6025 -> 5589; GPT-2, ResNet-50 and the odd sizes as before).
template <typename Begin>
constexpr uint32_t entry_of(uint32_t b, uint32_t first, uint32_t last, Begin begin) {
    while (first < last) {
        const uint32_t mid = (first + last + 1) >> 1;
        if (begin(mid) <= b) first = mid; else last = mid - 1;
    }
    return first;
}

// Which part of a tensor a wavefront of a workgroup handles, in units of what a wavefront handles.  A tile is what the `waves`
// wavefronts of one workgroup handle; consecutive workgroups run on different XCDs.  With a tile in one piece, each XCD asks for pieces
// of 2 to 16 KB of a stream at a time.  Memory is faster the finer consecutive bytes are spread over the XCDs (a stream's addresses go
// round its channels every few KB), so the tiles of a whole group of kTileGroup are dealt out: first the first wavefronts of all its
// workgroups, then the second ones, and so on.  In a tensor's last, incomplete group every tile is in one piece.  Only if all workgroups
// of a group go by this is every part of it handled once: whether they do is decided per call, not per launch, since a launch may end within a
// group (for_each_step_segment).  The traffic of a step
// without arithmetic over 2^30 elements, 256 lanes, in TB/s, in one piece -> groups of 8 / 16 / 32 / 64 / 128 tiles: AdamW 5.9 -> 6.3 / 6.5 /
// 6.6 / 6.65 / 6.3; plain FP32 AdamW 5.75 -> 6.3 (8), 6.8 (64), as single wavefronts 6.76.  The steps themselves: step_dealt.  What it
// costs: a line of scales serves several parts, each on another XCD, and every L2 fetches it (SGD: 1.85 % of the traffic; two or four consecutive
// parts on one XCD save that but are slower, a Llama layer Lion 334 -> 339 / 345 us).
constexpr int64_t kTileGroup = 32;
constexpr int64_t wave_part(int64_t tile, int64_t wave, int64_t waves, int64_t full_tiles) {
    const int64_t group = tile & ~(kTileGroup - 1);
    return group + kTileGroup <= full_tiles ? group * waves + wave * kTileGroup + (tile - group) : tile * waves + wave;
}

// A HIP launch must stay below 2^32 work-items (gridDim.x * blockDim.x), so work of more workgroups goes out as
// consecutive launches: of `total` workgroups of `threads` lanes each, those from `first` on that go with one launch.
constexpr int64_t kMaxWorkItems = ((int64_t)1 << 32) - 1;
constexpr int64_t launch_span(int64_t total, int64_t first, int threads) {
    const int64_t most = kMaxWorkItems / threads;
    return total - first < most ? total - first : most;
}

// The word of device memory by which the check of an unpack admits the copy behind it on the same stream.  Calls use a word one
// after the other, with ascending tickets from 1 on (whatever it holds before the first).  A copy that was not admitted has run
// before the call after it begins; one that was admitted may run at any later time, whatever calls on other streams have written by
// then: a refusal leaves the word high enough for all of them.
constexpr uint64_t verdict_word(uint64_t ticket, bool admitted) { return admitted ? ticket : ticket - 1; }
constexpr bool verdict_admits(uint64_t word, uint64_t ticket) { return word >= ticket; }

// How a workgroup hands its two sums to a host that watches: as four words of memory that the host reads, each half a sum and the ticket
// of the call.  A word is written at once, so that whoever finds the ticket in all four has both sums; nothing has to be ordered,
// fenced or cleared.  A call's ticket differs from those that the words can hold from calls before it.
constexpr int kNmseWords = 4;
constexpr uint64_t nmse_word(uint32_t half, uint32_t ticket) { return (uint64_t)ticket << 32 | half; }
constexpr bool nmse_ready(const uint64_t (&w)[kNmseWords], uint32_t ticket) {
    return (uint32_t)(w[0] >> 32) == ticket && (uint32_t)(w[1] >> 32) == ticket && (uint32_t)(w[2] >> 32) == ticket &&
           (uint32_t)(w[3] >> 32) == ticket;
}
// The bits of sum 0 or 1.
constexpr uint64_t nmse_sum(const uint64_t (&w)[kNmseWords], int i) { return (w[2 * i] & 0xffffffffu) | w[2 * i + 1] << 32; }

}  // namespace fo
#endif
