// Internal: types shared by the host side of the library (flashoptim_api.hip) and its
// device code (flashoptim_kernels.hip).  Not part of the public ABI.
#ifndef FLASHOPTIM_DEVICE_H
#define FLASHOPTIM_DEVICE_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "flashoptim_launch.h"

namespace fo {

constexpr int kGroup = 32;                         // quantisation group (Algorithms 2, 3)
constexpr int kThreads = 256;                      // lanes per workgroup (quantisers, sweep, self-test)
// Launch shapes of the step kernels: consecutive elements per lane and lanes per workgroup.  One workgroup handles one
// tile of chunk_elems() consecutive elements.
//   kUsual: eight elements per lane and 256 lanes.
//   kSmall: calls over fewer than kSmallElems elements fill less than half the chip with tiles of 2048: they take four
//       elements per lane, twice the workgroups with half the work per lane (kernel time, eight -> four elements per lane: a
//       flat tensor of 2^18 elements AdamW 3.9 -> 3.5 us, SGD 3.5 -> 2.8; 25 tensors of odd sizes below 2^16, SGD 4.9 -> 3.8;
//       at 2^20 elements the two are equal, from 2^22 on the larger tile wins by 2-8 %).
//   kWide: SGD and Lion over kWideElems elements or more, eight elements per lane and 512 lanes, three workgroups to a compute
//       unit (below); against kUsual, six to a unit, SGD: a Llama layer 345.0 -> 339.8 us, flat 2^27 209.5 -> 206.5, 400 M 632.8 ->
//       621.3, four layers 1394 -> 1394, with embedding and head 3058 -> 3045; GPT-2 201.9 with kUsual, 203.5 with kWide, 24 M
//       elements 39.4, 40.0.  Lion goes with SGD and is as fast either way: a layer 348.8 -> 343.2, 2^27 209.7 -> 212.6, 400 M
//       629.1 -> 636.1, four layers with embedding and head 3054 -> 3048.
// The ablation variants (weights not split, states not quantized, or both) move FP32 arrays: four elements per lane,
// so that a wavefront's 128-bit FP32 access covers whole cache lines (with eight, each of two accesses covered half
// of every line: the plain FP32 AdamW step over a decoder layer of Llama-3.1-8B, 218 M parameters, took 1034 us
// against 963 with four).  The plain FP32 step has no decode tables to stage, so its workgroups are single wavefronts
// that start and retire on their own (same layer, with 256 / 128 / 64 lanes: AdamW 974 / 955 / 928 us, SGD 639 / 629 / 599).
enum class StepShape { kSmall, kUsual, kWide };
constexpr int64_t kSmallElems = (int64_t)1 << 20, kWideElems = (int64_t)1 << 27;
constexpr StepShape step_shape(int kind, bool split, bool quant, int64_t elems) {
    if (!(split && quant)) return StepShape::kUsual;
    return elems < kSmallElems ? StepShape::kSmall : kind != 0 && elems >= kWideElems ? StepShape::kWide : StepShape::kUsual;
}
constexpr int step_vec(bool split, bool quant, StepShape shape) {
    return split && quant && shape != StepShape::kSmall ? 8 : 4;
}
constexpr int step_threads(bool split, bool quant, StepShape shape) {
    return shape == StepShape::kWide ? 512 : split || quant ? 256 : 64;
}
constexpr int chunk_elems(bool split, bool quant, StepShape shape) {
    return step_threads(split, quant, shape) * step_vec(split, quant, shape);
}

// How many workgroups of a launch share a compute unit.  The memory system is fastest with about 10 MB of loads on their
// way, which is what latency times bandwidth asks for; all that the registers admit (eight wavefronts per SIMD) have up to
// 25 MB on their way, queue up in front of the DRAM and make it change rows more often.  (Wavefronts that also compute for a
// while have fewer on average: the compressed steps want more of them than the FP32 ones.)  A launch is held to fewer by the
// LDS it asks for beyond what it uses.  The lines are where the best counts lie, in us with no limit -> with it:
//   AdamW, 6 of 256 lanes: Llama layer 442 -> 428, four layers with embedding and head 3994 -> 3867, flat 16 M 34.8 -> 34.5;
//       7 for lists of fewer than 2^27 elements, whose workgroups spend a larger part of their time on looking up their tile
//       (no more than two runs of one build differ by, but the same way in every list: with 6 -> 7 GPT-2 254.4 -> 253.5,
//       ResNet-50 54.1 -> 54.0, 60 tensors of 60 M 123.9 -> 122.4, 24 of 72 M 147.9 -> 146.3).  With 5: 4 layers 3856, GPT-2
//       248.1 (6: 244.7), ResNet-50 54.7.
//   SGD and Lion, 6 of 256 lanes or 3 of 512; before, four of 512 (all that fit): Llama layer 346 -> 341 / 345 -> 341, flat
//       400 M SGD 659 -> 637, GPT-2 200.8 -> 197.3 / 194.5 -> 194.1, ResNet-50 SGD 42.7 -> 42.2.
//   Plain FP32 steps, single wavefronts: AdamW 11 (Llama layer 896 -> 845, flat 25 M 104.2 -> 97.7, 300 M 1247 -> 1155; 32
//       fit), SGD and Lion 14 (603 -> 581, 69.3 -> 67.0, 829 -> 798).
//   Weight split only, 256 lanes: AdamW 4 (897 -> 832, 96.6 -> 93.8), SGD and Lion 5 (25 M 62.6 -> 62.1, 124 M 313.9 -> 303.6).
//   State quantisation only: AdamW 6 of 256 lanes (before, all of 512: 488 -> 484, 58.5 -> 56.9), SGD and Lion 7 (25 M 47.8
//       -> 47.6, 300 M 568 -> 546).
// Not held back: compressed steps of up to 2^22 elements, which are one generation of eight workgroups to a unit (2^22 elements in
// the caches: AdamW 9.58 us, with the limit 10.48, SGD 7.60, 7.96, Lion 7.29, 8.22; AdamW over 3 M 8.75, 8.92), and the
// ablation variants where stores do not go through (plain FP32 SGD over 5 M elements 15.3 us, with 18 wavefronts 16.4).
// A held launch leaves little of a unit's LDS to kernels on other streams (six workgroups: 2.5 KB).  No cost of that was found: two
// Llama layers of release calls on one stream beside bf16 products on another, until both are done, no limit -> limit: AdamW and
// ten products of 4096^3 2.02 -> 2.00 ms, three of 8192^3 3.37 -> 3.36, forty of 2048^3 2.00 -> 1.97; SGD 1.77 -> 1.77,
// 3.13 -> 3.13, 1.67 -> 1.69.
constexpr int kNoLimit = 0;
constexpr int step_resident(int kind, bool split, bool quant, StepShape shape, bool direct, int64_t elems, bool through) {
    if (split && quant && elems <= ((int64_t)1 << 22)) return kNoLimit;
    if (split && quant) return shape == StepShape::kWide ? 3 : kind == 0 && !direct && elems < ((int64_t)1 << 27) ? 7 : 6;
    if (!through) return kNoLimit;
    return split ? (kind == 0 ? 4 : 5) : quant ? (kind == 0 ? 6 : 7) : kind == 0 ? 11 : 14;
}
// Layout conversions, in us.
//   To FP32, 256 lanes, tiles dealt out (below): of AdamW's state 4 (with 4 / 5 / 6 / 8, flat 300 M 798 / 808 / 814 / 820, a Llama layer
//       571 / 579 / 580 / 589, GPT-2 326.5 / 329.2 / 328.4 / 334.0, flat 40 M 105.8 / 106.8 / 107.3 / 108.7), but 6 for lists of fewer than
//       2^26 elements (60 tensors of 60 M 159.6 / 157.7 / 156.1 / 157.0), where the two are within 1 % of each other on either side (with 4 / 6, 60
//       uneven tensors of 40 M 108.7 / 107.4, 60 M 161.1 / 159.4, 72 M 191.3 / 191.4, 90 M 238.5 / 237.0; 20 of them 107.6 / 107.1, 160.4 / 159.9,
//       190.0 / 191.4, 240.6 / 240.8); of the others' 6 (GPT-2 257 / 235 / 228 / 226, flat 300 M 591 / 546 /
//       545 / 543).  In one piece: 7 / 6 / 5 workgroups 5 M 15.8 / 15.8 / 15.9; under 2^22 elements no limit (2 M 6.5).
//   From FP32, single wavefronts: 20 for lists (with 18 / 20 / 22, AdamW GPT-2 321.9 / 318.9 / 329.0, a layer 563.7 / 559.8 / 581.8, 60 tensors of
//       60 M 157.4 / 154.8 / 155.9; SGD 229.8 / 222.7 / 224.1, 404.9 / 392.9 / 397.2, 113.9 / 110.9 / 108.8), 18 for a single tensor (AdamW 300 M
//       766.7 / 785.6 / 803.4, 200 M 510 / 525 / 541, 40 M 104.4 / 105.0 / 107.1; SGD 532 / 537 / 548, 354 / 356 / 368, 74.2 / 73.6 / 74.4), of which
//       those of SGD and Lion up to 60 M would be 1 % faster with 20 (34 M 62.9 / 62.1, 60 M 108.5 / 107.3, 100 M 178.7 / 179.1; AdamW 34 M 89.1 /
//       88.5, 60 M 154.5 / 156.8).
constexpr int convert_resident(bool compress, bool has_v, bool direct, bool through, int64_t elems) {
    if (compress) return !through ? kNoLimit : direct ? 18 : 20;
    if (elems < ((int64_t)1 << 22)) return kNoLimit;
    return through && has_v && (direct || elems >= ((int64_t)1 << 26)) ? 4 : 6;
}
// The dynamic LDS, in bytes, with which exactly `resident` workgroups that use `used` bytes fit into a compute unit's
// 160 KB (given out in units of 1280 bytes).
constexpr unsigned lds_to_hold(int resident, unsigned used) {
    return resident == kNoLimit ? 0u : (128u / (unsigned)resident) * 1280u - used;
}

// Whether the stores of a call go through to memory at device scope, or stay non-temporal only.  Lines that are passed on
// as they are written leave the DRAM fewer, larger turns from reading to writing and the end of the kernel nothing to write
// back.  But lists whose arrays fit the 256 MB memory-side cache with room to spare are faster where their lines may wait.
// In us, non-temporal -> through:
//   steps, in place, by the size of their arrays: plain FP32 AdamW over a Llama layer (3 GB) 851 -> 839, SGD 619 -> 584, four
//       Llama layers AdamW (14 GB) 3942 -> 3890, one by gradient release 453 -> 450, GPT-2 Lion (0.8 GB) 195.3 -> 194.1, AdamW
//       over 60 M elements (430 MB) 123.5 -> 122.0, ResNet-50's 25.6 M (182 MB) 54.8 -> 54.3; 24 M (171 MB) 50.5 -> 50.3,
//       FP32 AdamW over 12 M (168 MB) 51.1 -> 52.1, SGD over 24 M (145 MB) 39.5 -> 40.1, AdamW over 6 M (43 MB) 16.9 -> 17.2;
//   conversions: GPT-2 compress 339.7 -> 336.2, decompress 342.8 -> 341.8; 25 M elements 70.6 -> 70.4 and 70.6 -> 71.4, 12 M
//       33.7 -> 34.2 and 35.2 -> 35.7;
//   codecs, the six of them: 38.6 M elements 215.7 -> 212.1, 12 M 78.4 -> 76.8, 5 M 40.7 -> 40.9.
constexpr int64_t kThroughBytes = (int64_t)168 << 20;
constexpr int step_array_bytes(int kind, bool split, bool quant) {      // per element, without the scales
    return 2 + (split ? 3 : 4) + (kind == 0 ? 2 : 1) * (quant ? 1 : 4);
}
constexpr bool step_through(int kind, bool split, bool quant, int64_t elems) {
    return elems * step_array_bytes(kind, split, quant) >= kThroughBytes;
}
// Whether the tiles of a call are dealt out among wavefronts (wave_part): where stores go through and there is more than one
// wavefront to a workgroup, but not for AdamW with quantised states, compressed or not.  That one is bound by the package's power and its
// instructions; dealt out it is slower (compressed, four Llama layers with embedding and head 3855 -> 3902 us, a layer 447 -> 454, GPT-2 254.5 ->
// 259.5, though on a card with some power to spare two layers took 868 -> 848; state quantisation only, the whole Llama list 17785 -> 18105, a
// layer 484.3 -> 489.6, GPT-2 277.7 -> 278.8).  The others, in one piece -> dealt out, in us: SGD two Llama layers 689 ->
// 657, flat 400 M 629 -> 606, GPT-2 198.6 -> 187.9, 24 tensors of 72 M 112.7 -> 110.0; Lion 688 -> 662, 620 -> 603, 199.4 -> 187.3,
// 113.0 -> 110.3; weight split only, a layer, AdamW 822 -> 782, SGD 532 -> 507, Lion 534 -> 513, 25 M 94.9 -> 90.2, 62.7 -> 60.1, 62.9 -> 60.4; state
// quantisation only, SGD the whole list 14695 -> 14681, a layer 399.2 -> 399.5, GPT-2 230.7 -> 227.6, Lion 14743 -> 14680, 400.6 -> 399.1, 232.3 ->
// 228.1.  Calls whose stores do not go through are 1-2 % slower dealt out (SGD over 10 M elements 16.8 -> 17.0 us).
constexpr bool step_dealt(int kind, bool split, bool quant, bool through) {
    return through && (split || quant) && !(kind == 0 && quant);
}
// Conversions to FP32 are dealt out where their stores go through (in one piece -> dealt out, with the limits above on both sides, AdamW
// GPT-2 341.0 -> 326.5 us, a Llama layer 609.6 -> 571.0, flat 300 M 822 -> 798, 40 M 110.0 -> 105.8; SGD 237.5 -> 228.0, 413.1 -> 399.7,
// 561 -> 545, 76.6 -> 73.4).  Those from FP32 are single wavefronts.  The quantisers and dequantisers are 1 to 5 % slower dealt out.
constexpr bool convert_dealt(bool compress, bool through) { return !compress && through; }
// (Of the whole call.  Beyond 2^38 elements the single wavefronts that go with it would be more than a 31-bit index counts.)
constexpr bool convert_through(int64_t elems) { return elems >= ((int64_t)1 << 25) && elems < ((int64_t)1 << 38); }
constexpr bool codec_through(int64_t elems) { return elems >= ((int64_t)1 << 23); }

constexpr int kCopyPiece = 16 * 1024;        // checkpoint copy: bytes per workgroup
constexpr int kHeaderStepAt = 16;            // byte offset of the step (little-endian int64) in a blob's header

// One tensor as the kernels see it (device pointers), 104 bytes.
struct TensorDev {
    void* param;
    int8_t* rho;
    const void* grad;
    int8_t* m_q;
    uint16_t* m_scale;
    uint8_t* v_q;
    uint16_t* v_scale;
    float* theta32;   // ablation variants: FP32 master weight (weights not split)
    float* m32;       // ablation variants: FP32 momentum (states not quantized)
    float* v32;       // ablation variants: FP32 variance
    int64_t numel;
    float lr, wd;
    uint32_t first_tile;   // multi-tensor launch: index of the workgroup that handles the tensor's first tile
    uint32_t n_tiles;      // multi-tensor launch: number of tiles (workgroups) of the tensor
};

// Per-call scalars, computed once on the host.
// Operand range of the short divisions of the AdamW kernels (numerator, denominator and eps inside it).
constexpr float kDivFastLo = 8.673617379884035e-19f;    // 2^-60
constexpr float kDivFastHi = 1.152921504606847e18f;     // 2^60

struct StepConsts {
    float beta1, beta2;   // AdamW/Lion betas; SGD: beta1 = momentum
    float omb1, omb2;     // 1.0f - beta (FP32 subtraction)
    float rbc1, rbc2;     // 1.0f / (float)(1 - beta^t), AdamW only
    float eps;
    float k255_hi, k255_lo;   // 255 * sqrt(1 / rbc2) in double, as two floats: used only to pre-estimate variance codes
    float v_max, m_max;   // largest v_t and |m_t| for which the short square root and division serve: 2^60 / rbc2 and
                          // 2^60 / rbc1 rounded down, or -1 when eps is outside [2^-60, 1] (the kernels then use
                          // sqrtf and the IEEE division throughout)
    float sqrt_min;       // smallest v_t for the same: 2^-96, or +inf while the short square root has not passed its
                          // check on this device; the step kernels fill it in from StepArgs::sqrt_min_word
};

// One logical launch is issued as consecutive launches that cover at most this many elements each.
// Measured on the Llama list (8.03 G parameters): the memory-bound SGD and Lion steps run 3-9 % faster
// in ~30-60 launches than in one launch of 1.96 M workgroups (12.9-13.0 vs 13.4-14.0 ms); AdamW gains
// under 1 % and loses with segments below 64 M elements; below ~25 K workgroups per launch the gaps
// between launches take the gain back.
#ifndef FO_SEGMENT_ELEMS
#define FO_SEGMENT_ELEMS (1 << 28)
#endif
constexpr int64_t kSegmentElems = FO_SEGMENT_ELEMS;
// launch_part(first, n) for each of these launches: the tiles first .. first + n - 1 of the call's `tiles`, up to the first that fails.
template <typename F>
hipError_t for_each_segment(int64_t tiles, int64_t tile_elems, F launch_part) {
    const int64_t most = kSegmentElems / tile_elems > 0 ? kSegmentElems / tile_elems : 1;
    for (int64_t first = 0; first < tiles; first += most) {
        const hipError_t e = launch_part(first, tiles - first < most ? tiles - first : most);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
// The same for a step, launch_part(first, n, through).  One decision for the whole call: it is also that on which wavefront handles
// what (step_dealt), and of the tiles that wave_part deals out together some may lie in one launch and some in the next.
template <typename F>
hipError_t for_each_step_segment(int kind, bool split, bool quant, int64_t tiles, int64_t tile_elems, F launch_part) {
    const bool through = step_through(kind, split, quant, tiles * tile_elems);
    return for_each_segment(tiles, tile_elems, [&](int64_t first, int64_t n) { return launch_part(first, n, through); });
}
struct StepArgs {
    TensorDev* tensors;         // device table (multi-tensor launch)
    const uint32_t* coarse;     // device table: tensor index per 2^coarse_shift workgroups (flashoptim_launch.h)
    uint32_t coarse_shift;
    uint32_t block_offset;      // tile index of this launch's workgroup 0 (a list or tensor is covered by several launches)
    // A new learning rate that all tensors of a multi-tensor step share travels here instead of in an update of the table,
    // so that a schedule, which changes it with every step, has no launch in front of every step (AdamW, with and without
    // it: ResNet-50 list 54.7 and 52.3 us a step, GPT-2 237.3 and 235.1, 25 odd sizes 9.3 and 5.8).  The rate in use is (table's bits & table_lr_mask) |
    // shared_lr_bits: the mask is 0 for a new rate, otherwise all ones beside bits of 0.  The workgroup of a tensor's
    // first tile writes a new rate into the table behind it, for launches that read it there: captured ones, above all.
    uint32_t table_lr_mask;
    uint32_t shared_lr_bits;
    TensorDev single;           // the one tensor of a direct launch
    bool through;               // stores go through to memory (step_through, convert_through; the same for all launches of a call)
    StepConsts c;
    const float* sqrt_min_word; // AdamW steps: device word that holds StepConsts::sqrt_min for this device
};

struct CopySegment {
    const uint8_t* src;
    uint8_t* dst;
    int64_t bytes;       // bytes to copy
    int64_t pad_bytes;   // >= bytes; [bytes, pad_bytes) of dst is zero-filled
    uint32_t first_piece;   // index of the workgroup that copies the segment's first piece
    uint32_t n_pieces;
};

struct CopyArgs {
    const CopySegment* segs;
    const uint32_t* coarse;     // segment index per 2^coarse_shift pieces, as in StepArgs
    uint32_t coarse_shift;
    uint32_t n_pieces;
    uint32_t piece_offset;      // index of this launch's workgroup 0
    // packing: the blob's header and table (nullptr: none), which one further workgroup writes to header_dst with `step`
    // in its place
    const uint4* header;
    uint4* header_dst;
    uint32_t header_n16;
    int64_t step;
    const uint64_t* verdict;    // unpacking: the word that says whether the blob belongs to this list (nullptr: no such
    uint64_t ticket;            // condition), and the ticket of this call (verdict_admits)
};
// Unpacking a blob with a short table: every workgroup compares `header`, what the list expects, with `found`, the blob's own.  The first
// tells the host: out[0] becomes 1 or 0 and out[1] the blob's step, then *flag (all pinned) the ticket's low half.
struct CheckedCopyArgs : CopyArgs {
    explicit CheckedCopyArgs(const CopyArgs& a) : CopyArgs(a) {}
    const uint4* found;
    int64_t* out;
    uint32_t* flag;
};

hipError_t launch_step(int kind, bool direct, bool split, bool quant, StepShape shape, bool exact, const StepArgs& a,
                       int64_t n_blocks, hipStream_t s);
// Lanes per workgroup and elements per tile of the layout conversions.  Compressing stages nothing: calls whose stores go
// through take single wavefronts (GPT-2 344.8 -> 322.6 us, 300 M elements 816 -> 777, 25 M 70.0 -> 69.8);
// smaller ones 256 lanes (5 M 15.0 us, as single wavefronts 15.5).  Decompressing takes 256 (GPT-2 340.0 us, 128 lanes 343.9, single
// wavefronts 346.9; 300 M 834, 862 and 842).
constexpr int convert_threads(bool compress, bool through) { return compress && through ? 64 : 256; }
constexpr int convert_chunk(bool compress, bool through) { return convert_threads(compress, through) * 4; }
hipError_t launch_convert(bool has_v, bool compress, bool direct, const StepArgs& a, int64_t n_blocks, hipStream_t s);
hipError_t launch_probe(int kind, bool direct, StepShape shape, const StepArgs& a, int64_t n_blocks, hipStream_t s);
hipError_t launch_split(int bits, const float* theta, void* param, void* rho, int64_t n, hipStream_t s);
hipError_t launch_reconstruct(int bits, const void* param, const void* rho, float* theta, int64_t n, hipStream_t s);
constexpr int kSweepStats = 8 + 3 * 256;
hipError_t launch_clock_monitor(unsigned long long* samples, int n_samples, unsigned long long ticks_per_sample,
                                hipStream_t s);
hipError_t launch_sweep(int bits, bool directional, uint64_t first, uint64_t stride, uint64_t count, double* stats,
                        hipStream_t s);
hipError_t launch_quantize(bool variance, bool linear, const float* x, void* q, uint16_t* scale, int64_t n, hipStream_t s);
hipError_t launch_dequantize(bool variance, bool linear, const void* q, const uint16_t* scale, float* x, int64_t n,
                             hipStream_t s);
constexpr int kNmseThreads = 512, kNmseMaxBlocks = 1024;
int nmse_blocks(int64_t n);
// words: kNmseWords words of pinned memory for each of the nmse_blocks(n) workgroups, its sums with this call's ticket (nmse_word)
hipError_t launch_nmse(bool variance, bool linear, const float* x, int64_t n, uint64_t* words, uint32_t ticket, hipStream_t s);
hipError_t launch_copy(CopyArgs a, hipStream_t s);
// The blobs whose unpacking takes that way: every workgroup, for 16 KB of its own, reads header and table twice (the list's and the blob's), so
// they are short (252 tensors), and the launch that it saves is worth what the barrier costs.  Smaller ones are bound by the wait for the
// verdict, which a kernel of its own reaches sooner.  In us, a kernel ahead of the copy -> checked by every workgroup, a pack and an unpack, few tensors:
// 5 MB 15.8 -> 16.8, 15 MB 20.4 -> 20.7, 33 MB 26.6 -> 24.3, 103 MB 68.5 -> 64.1, 205 MB 133.9 -> 130.0; an unpack: ResNet-50's 131 MB 46.3 -> 45.1,
// 512 MB 163.0 -> 163.3, GPT-2's 638 MB 193.6 -> 195.9, 1.5 GB 456 -> 462.  An unpack of 28 / 101 / 244 MB by the tensors in its table: 60 of them
// 13.7 -> 12.6, 35.3 -> 34.4, 79.4 -> 77.9; 200 15.0 -> 13.9, 35.9 -> 35.5, 80.4 -> 80.1; 252 14.2 -> 14.4, 37.1 -> 37.3, 81.6 -> 81.2; 330 16.4 -> 15.2,
// 36.4 -> 37.3, 82.2 -> 81.6; 500 14.9 -> 16.0, 38.7 -> 40.2, 82.1 -> 83.8; 1020 25.2 -> 25.0, 48.0 -> 49.0, 84.6 -> 97.0.
constexpr int64_t kCheckedHeader = 4096;
constexpr bool checked_copy(int64_t blob_bytes, int64_t header_bytes) {
    return blob_bytes >= (int64_t)24 << 20 && blob_bytes <= (int64_t)256 << 20 && header_bytes <= kCheckedHeader;
}
hipError_t launch_checked_copy(CheckedCopyArgs a, hipStream_t s);
// Moves `bytes` (rounded up to 16: both buffers must have room) from pinned host memory to device memory.
hipError_t launch_move(const void* src, void* dst, size_t bytes, hipStream_t s);
// Compares the header and table at `blob` with the expected ones, the step apart: *verdict (device) becomes verdict_word of the
// result, out[0] (pinned) 1 or 0, out[1] the blob's step; *flag (pinned) becomes the ticket's low half once they are there.
hipError_t launch_check_header(const void* expected, const void* blob, size_t bytes, uint64_t* verdict, int64_t* out,
                               uint32_t* flag, uint64_t ticket, hipStream_t s);
// New values for `count` entries of a step's table, from entry `first` on.  Only the fields of the entries that change
// travel, in the order of the masks below, so that as many entries as possible go with one launch.
enum : uint32_t { kUpdateGrad = 1, kUpdateLr = 2, kUpdateWd = 4 };
constexpr uint32_t update_words(uint32_t fields) {
    return ((fields & kUpdateGrad) ? 2 : 0) + ((fields & kUpdateLr) ? 1 : 0) + ((fields & kUpdateWd) ? 1 : 0);
}
struct TableUpdate {
    uint32_t first, count, fields;
    uint32_t words[960];        // update_words(fields) of them per entry
};
constexpr uint32_t update_batch(uint32_t fields) { return (uint32_t)(sizeof(TableUpdate::words) / 4) / update_words(fields); }
static_assert(sizeof(TableUpdate) + 2 * sizeof(void*) <= 4096, "kernel arguments");
hipError_t launch_table_update(const TableUpdate& u, TensorDev* table, hipStream_t s);
constexpr int kSelftestSectionCount = 7;
constexpr unsigned long long kSelftestSqrtValues = 0x7f800000ull - 0x0f800000ull;   // section 2: every FP32 value in [2^-96, FLT_MAX]
constexpr int kSelftestCounters = 15;   // two per section, then the inexact count of section 6
// Section 4 (variance codes) runs once per (beta2, step, group scale): steps 1..20, then 50, 100, 200, 500, ... 10^6.
constexpr int kSelftestVarSteps = 34;
constexpr int64_t selftest_var_step(int i) {
    if (i < 20) return i + 1;
    const int j = i - 20;                        // 50, 100, 200, 500, 1000, ... (j = 0 .. 13)
    const int64_t lead[3] = {5, 10, 20};
    int64_t p = 10;
    for (int k = 0; k < j / 3; ++k) p *= 10;
    return lead[j % 3] * p;
}
static_assert(selftest_var_step(19) == 20 && selftest_var_step(20) == 50 && selftest_var_step(21) == 100 &&
              selftest_var_step(22) == 200 && selftest_var_step(33) == 1000000, "");
hipError_t launch_selftest(unsigned long long* counters, int section, const StepConsts& c, float scale_r,
                           hipStream_t s);

}  // namespace fo
#endif
