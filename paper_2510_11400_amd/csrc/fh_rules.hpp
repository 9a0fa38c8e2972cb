// Rules by which the host chooses the shape of a launch, apart from the launches so that they can be looked at on any
// machine: plain C++, no HIP.
#pragma once

#include <stdint.h>

namespace fh {

// The classification's count pass where it has value ranges.
// A workgroup sends a histogram of `channels` counters to the tensor's own, and on wide tensors those atomics are what
// the pass takes, so a launch with such a tensor has workgroups of eight waves that share one.  With four, 100 MB of
// 3072 channels take 26.4 us (fp32) and 33.6 us (bf16), with eight 23.0 and 28.6, 768 channels 28.7 and 42.1, then 22.9
// and 28.3; narrow tensors are better off with four (16 MB to 557 MB of feature maps: up to 4 us of 27).
inline int marked_waves_per_workgroup(int64_t widest) { return widest > 512 ? 8 : 4; }

// Spans of 1024 elements per wave, of a tensor of `tensor_spans` with `channels` channels in a launch of `launch_spans`
// altogether and `widest` channels at most.  A wave reads its pieces one batch after the other, so a launch is cut into 4096 waves (four per SIMD) before a wave
// gets a second span: with eight spans a wave whatever the size, 4 MB took 9.9 us and 64 MB 14.0 us where most pieces hold
// an outlier; this way 4.4 and 12.7 (where few do, 4.3 and 6.7, now 3.7 and 6.0).  A wide tensor is cut into 256 workgroups at most
// until a wave has its fill (25 MB of 768 channels in workgroups of four waves: 13.3 us with six spans, 15.2 with three,
// 25.5 with one).  Eight spans are as many as a wave looks at together.
inline int32_t marked_spans_per_wave(int64_t launch_spans, int64_t tensor_spans, int64_t channels, int64_t widest)
{
    int64_t spans = launch_spans / 4096;
    const int64_t least = tensor_spans / (256 * marked_waves_per_workgroup(widest));
    if (channels > 512 && least > spans) spans = least;
    return (int32_t)(spans < 1 ? 1 : spans > 8 ? 8 : spans);
}

// Tiles in runs.  Workgroups are dealt to the eight XCDs one by one.  Here a window of 8 * RUN of them takes as many tiles so that each XCD has RUN
// consecutive ones, the windows following one another: what a launch has touched at any time is still one stretch of
// memory, so that the codes written last are the ones that the restore begins with finds in the memory-side cache.
// (With one window, an eighth of the launch to each XCD, the quantiser gained and the restore lost as much.)  The last workgroups,
// short of a window, stay where they are.  (Host and device: a constexpr function is both.)
constexpr uint32_t kXcds = 8;
template <uint32_t RUN> constexpr uint32_t tile_in_run(uint32_t block, uint32_t blocks)
{
    constexpr uint32_t kWindow = kXcds * RUN;
    const uint32_t first = block / kWindow * kWindow, at = block - first;
    return first + kWindow <= blocks ? first + at % kXcds * RUN + at / kXcds : block;
}
// Whether the tiles of the plain quantiser of fp32 and of the restore to fp32 go to the XCDs in runs, in a launch of `tiles`: 16 KiB of input
// each, respectively 8 KiB of fp32 output.  The quantiser gains in fp32 from some 200 MB on: with runs of 128 a plan's 2 GiB both
// ways 868 -> 819 us, 1 GiB 398 -> 390, 240 MB of feature maps 89.5 -> 88.4; 278 MB 103.4 and 103.0, 60 MB 26.5 and 27.0; bf16 loses
// (encoder set 398 -> 407).  The restore of fp32 with runs of 64: encoder set 398 -> 379 us, 126 MB of it 41.0 -> 39.1, the plan
// 868 -> 854, MobileNetV2-style set 201 -> 197, 60 MB 26.5 and 26.3; runs of 32 gain a half of that, of 128 as much.  By the codes'
// width, restore in order and in runs, codes and output in the cache | from sets in turn, 1.6 GB of them:
//   2 bits 67 MB 11.2 and 11.3 | 11.3 and 11.6, 101 MB 16.8 and 16.8 | 16.9 and 16.6, 168 MB 28.3 and 27.3 | 28.3 and 26.2, 557 MB 97 and 87 | 97 and 87;
//   4 bits 67 MB 11.4 and 11.5 | 11.8 and 12.2, 101 MB 17.0 and 16.8 | 17.0 and 17.5, 168 MB 28.1 and 27.0 | 27.5 and 27.6, 557 MB 92 and 86 | 92 and 87;
//   8 bits 67 MB 11.1 and 13.5 | 15.2 and 15.8, 101 MB 16.4 and 17.7 | 20.8 and 22.3, 168 MB 30.2 and 30.6 | 32.0 and 33.2, 268 MB 47.2 and 47.4 | 53.4 and
//   53.2, 335 MB 58.9 and 58.9 | 65.6 and 65.8, 400 MB 70.0 and 70.2 | 80.0 and 78.4, 800 MB 139 and 138 | 159 and 155;
//   a third of each 84 MB 14.9 and 14.4 | 17.4 and 17.6, 134 MB 23.3 and 22.1 | 26.1 and 24.8, 268 MB 44.4 and 43.1 | 44.6 and 43.5.
// Both ways on sets in turn, 2 and 4 bits lose 0.4 us of 25 at 67 MB, 2 bits gain from 92 MB on, 4 bits from 200 MB on with nothing either way before;
// 8 bits 67 MB 28.5 and 29.0, 101 MB 40.4 and 41.2, 335 MB 128 and 128, 800 MB 314 and 306 (on one tensor again and again 67 MB 30.4 and 28.3,
// 84 MB 34.8 and 35.2).  So sets of mostly 8 bits wait for 335 MB.  Restoring bf16 gains nothing (280 to 286 us), nor do the routed forms.  (A kernel of its own each: the test in the others cost a set of 60 MB 0.3 us of 25.6.)
inline bool compress_in_runs(uint32_t tiles) { return tiles >= 12288; }
inline bool restore_in_runs(uint32_t tiles, uint64_t elements, uint64_t code_bits)
{
    return tiles >= (code_bits > 6u * elements ? 40960u : 8192u);
}

// Whether the routed quantiser or its restore takes one tensor's descriptor in a short argument segment (fh_batch.hpp).  One fp32 tensor,
// both ways, with the batch's arguments and with these, us: 0.8 MB 10.6 and 7.0, 3.2 MB 10.9 and 7.7, 19 MB 14.7 and 14.0.  Putting the
// descriptor together again costs scalar registers, and with them the 65th vector register of the bf16 form, so that seven
// waves fit a SIMD: launches that the device holds at once in workgroups of four such waves, and whose kernel is over before
// a longer one is enqueued.
inline bool one_by_itself(int32_t tensors, uint32_t tiles) { return tensors == 1 && tiles <= 256u * 7u; }

// How often a wave of a large launch looks at that many spans.  A workgroup's histogram of a wide tensor is 3072 counters to clear
// and to add in for the outliers of 64 spans; once there are waves for a whole round of the device (8192 of eight spans), twice the
// spans to a histogram save half of that, the ranges of the second eight on their way meanwhile.  Count pass of the 720 MiB
// encoder set 56 -> 45 us; classification of three tensors of 3072 channels (151 MB) 56 -> 50, of twelve 154 -> 144, three of 16384
// channels 154 -> 134; with 768 channels, whose histograms are short, 76 -> 77, feature maps 16 -> 20: these keep one.
inline int32_t marked_looks_per_wave(int64_t launch_spans, int64_t channels) { return channels > 1024 && launch_spans > 65536 ? 2 : 1; }

// Whether the count pass sets a tensor's mask as it adds to the counters, or a launch behind it does.  The additions are then waited for, and
// a wide tensor's workgroup has many: 3 tensors of 3072 channels 52 us with the launch and 56 without, 3 of 16384 128 and
// 154, 24 of 768 78 and 76, 18 of 1024 131 and 126, one of 768 17.9 and 16.9.
inline bool mask_with_the_counts(int64_t channels) { return channels <= 1024; }
// The same without value ranges, where more of a large tensor's workgroups add to a counter at a time.  768 channels: one fp32 tensor of
// 24 Mi elements 49.3 us with the launch and 54.1 without, two of 12 Mi 49.2 and 51.5, eight of 64 Mi (bf16) 445 and 464, 26 of 4 Mi 149 and
// 151, 26 of 1 Mi 49.3 and 48.2; 1024 channels, eight of 4 Mi (bf16) 36.7 and 34.6, one of 64 Mi 71.9 and 77.8.
inline bool mask_with_the_counts_unranged(int64_t channels, int64_t tensor_spans)
{
    return mask_with_the_counts(channels) && (channels <= 512 || tensor_spans <= 4096);
}
// The same where the limits are apart (limits_apart): waiting is then most of what a short workgroup does (eight bf16 tensors of
// 16 Mi elements without ranges 122 us with the launch and 137 without, of 128 Mi 949 and 1020; with ranges, one of 768 Mi with 256 channels
// 364 and 393).  Only a tensor alone, without ranges, is bound by the additions themselves, and the launch would come on top: 64 Mi
// 110.5 and 107.5, 1000 Mi 1575 and 1535 (64 channels), 64 Mi with 512 channels 55.9 and 54.3, 512 Mi 367 and 371.
inline bool mask_with_the_counts_apart(int64_t channels, bool ranges, int32_t tensors) { return !ranges && tensors == 1 && channels <= 512; }

// Whether a launch before the count pass finishes the moments, or the first wave of each of its workgroups does.  The launch: so many
// tensors and workgroups, `of_one_span` of these of tensors that have a span for each wave (without value ranges, up to 512 channels), one
// of which is `crowded` (its workgroups' additions meet on few counters).  The launches apart, this one and the one for the
// masks behind, take 3 us each; in the pass, the limits and the masks make every workgroup take longer.  Both in the pass and both apart, us:
//   with ranges: 16 tensors of 16 Mi elements (8192 workgroups) bf16 136 and 135, one of 256 Mi, 256 channels, 134 and 127, eight of 64 Mi (16384), 32
//   channels, 309 and 279, fp32 492 and 461, three of 256 Mi 537 and 480, 799 and 732; eight of 16 Mi (4096) 69 and 70, 114 and 116;
//   several without, fp32: two of 4 Mi (2048), 1 channel, 30.7 and 30.7, 64 channels 21.5 and 26.8; three of 4 Mi (3072), 3 channels, 41.9 and 35.1, 64
//   channels 25.6 and 29.9; 12 of 1 Mi (3072), 3 channels, 23.2 and 26.5; two of 8 Mi (4096), 16, 64 and 128 channels, 64.2 and 57.4, 40.6 and 37.7, 31.5
//   and 34.1; four of 4 Mi, 32 and 64 channels, 36.5 and 36.5, 31.2 and 34.1; 20 of 1 Mi (5120), 64 channels, 33.1 and 32.0, 26 of 1 Mi 43.5 and 41.0, eight
//   of 16 Mi bf16 141 and 122, of 128 Mi 1130 and 949;
//   one without: 20 Mi (5120), 64 channels, 44.1 and 47.0, bf16 38.9 and 41.7, 64 Mi, 512 channels, 89.5 and 94.7, bf16 60.1 and 55.7, 512 Mi bf16 459
//   and 367;
//   wide ones without: 16 of 16 Mi, 3072 channels, bf16 188 and 187, fp32 345 and 348, two of 12 Mi 33.5 and 36.8, 43.5 and 44.9.
inline bool limits_apart(bool ranges, int32_t tensors, uint32_t workgroups, uint32_t of_one_span, bool crowded)
{
    if (ranges) return workgroups >= 8192;
    if (tensors == 1) return of_one_span > 5120;
    return of_one_span >= 5120 || (of_one_span > 2048 && crowded);
}
inline bool counters_are_crowded(uint32_t workgroups, uint32_t channels) { return workgroups >= 1024 && workgroups / 32 >= channels; }

// Histogram workgroups of a stream of n symbols: four vectors per thread up to 4 Mi symbols, eight of what lies beyond, more in long
// streams, since a workgroup clears and adds up 32 KiB of counters whatever it counts.  (Eight throughout, the five streams of 8 MB
// of the whole chain take 7.5 us, this way 5.5.)  Where that is a few more than one for each compute unit, one for each: of 281 workgroups a
// tenth of the units has two, and all wait for these.  Encoding 31 MB of three symbols, index bytes, noise 40.4, 64.5, 52.0 us with the few more and
// 37.2, 61.1, 48.7 without, 33 MB 41.2, 52.6, 52.5 and 37.9, 49.2, 49.2; 36 MB (275, or 307) 47.7, 59.4, 59.8 and 48.1, 59.8, 59.9, 50 MB and more the same.
constexpr uint64_t kHistRound = 1024 * 16;                    // symbols that a workgroup takes at a time
constexpr uint32_t histogram_workgroups(uint64_t n)
{
    constexpr uint64_t four = 4u * kHistRound, eight = 8u * kHistRound, few = 64, units = 256, most = 2u * units;
    const uint64_t want = n == 0 ? 0 : n <= few * four ? n / four + 1u : few + (n - few * four) / eight + 1u;
    const uint64_t held = want <= units ? want : n / eight + 1u > units ? n / eight + 1u : units;
    return (uint32_t)(held < most ? held : most);
}

// The Huffman encoder's group sums in a launch of `groups` altogether: scanned by a kernel between the count and the write
// pass, or every workgroup of the write pass adds up those before its own.  Adding up saves that launch and makes every
// workgroup of the write pass take longer, so what counts is how many of those there are.  Encoding, scanned and not: one
// stream of 64 groups 36.9 and 36.3 us, of 1024 76.4 and 73.7, of 4096 203.4 and 200.8, of 6000 317 and 317, of 12288
// 599 and 609; 24 streams of 335 groups 394.5 and 395.7, 24 of 1024 1108 and 1124, six of 4096 1122 and 1151.
inline bool group_sums_are_scanned(int64_t groups) { return groups > 4096; }

// Is there a scan of the sums of a set's `groups` of tiles between the sparse stage's passes, in a launch of `of_launch` groups?  Without one each
// group adds up those before it, eight bytes for a group.  Encode | decode, scanned and not, us:
//   window 2, one set: 2100 groups 17.6 and 13.4 | 17.4 and 13.3, 4000 21.1 and 17.9 | 20.4 and 16.4, 6000 26.6 and 25.5 | 25.0 and 22.7, 8000 33.0
//   and 34.9 | 29.8 and 30.9; three of 2100 25.5 and 24.0 | 23.8 and 21.3, two of 4000 30.0 and 30.5 | 26.8 and 26.1, five of 2048 35.4 and 36.7 | 30.8
//   and 31.1, five of 4000 57.8 and 66.4 | 51.1 and 58.3;
//   window 4: 2100 25.8 and 22.8 | 21.8 and 17.7, 4000 39.1 and 37.1 | 28.2 and 25.8, 6000 51.0 and 50.0 | 38.5 and 37.1, 8000 63.4 and 64.6 | 47.7
//   and 48.7; two of 4000 60.2 and 60.9 | 44.4 and 44.6 (without a bound 60.1 and 59.0 | 51.9 and 44.9), five of 2048 76.8 and 80.4 | 51.8 and
//   52.5, five of 4000 138.9 and 152.8 | 90.4 and 99.5;
//   window 8, whose groups do the most: 2048 55.1 and 53.5 | 40.2 and 38.9, 2500 63.5 and 62.5 | 47.7 and 46.7 (without a bound 52.5 and 54.5 | 46.2
//   and 41.4), 3500 80.2 and 81.5 | 60.2 and 61.3, 4000 86.8 and 88.1 | 66.3 and 68.5, 6000 130 and 144 | 92 and 100.
// (Several small sets are added up in any launch: 24 of 1000, window 4, lose 8 of 167 and 7 of 106 us by it.)
constexpr uint32_t kMostAddedUp = 4096;
inline bool sparse_sums_are_scanned(uint32_t groups, uint32_t of_launch, int window)
{
    return groups > (window < 8 && of_launch <= 8192 ? kMostAddedUp : 2048u);
}

// The Huffman decoder's stores, in a call of `symbols`: whether half a cache line waits for its other half.
// Where the memory-side cache holds the output, half lines meet there, and storing early is better: the last stores of a
// pass are fewer (51 MB 41.4 us, 42.8 in whole lines; 268 MB of two bits a symbol 168 and 175).  Beyond, half lines reach
// memory: 1.6 GB were written as 2.1 and took 1018 us, in whole lines 945; two streams of 201 MB 260 and 252, three of 268 MB
// 523 and 491.
inline bool decode_in_whole_lines(uint64_t symbols) { return symbols >= (uint64_t)384 << 20; }

// The whole chain's maps, `bytes` in a call: whether the sparse stage leaves them in the memory-side cache for the restore.
// All maps of a call are written before the restore begins; beyond a part of the cache's 256 MB the first are gone when it
// reads them, and ordinary stores then only write back beside it.  Restore of feature maps, both stages, ordinary stores
// against stores that pass the caches by: fp32 34 MB 142 and 172 us, 85 MB 176 and 206, 132 MB 242 and 230, 157 MB 268 and
// 243; one tensor 77 MB 140 and 148, 154 MB 214 and 192; bf16 79 MB 214 and 250, 103 MB 276 and 278, 132 MB 336 and 328.
inline bool maps_stay_in_cache(uint64_t bytes) { return bytes <= (uint64_t)96 << 20; }

}  // namespace fh
