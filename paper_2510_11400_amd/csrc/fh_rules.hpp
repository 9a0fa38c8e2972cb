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

// Whether the tiles of the plain quantiser of fp32 and of the restore to fp32 go to the XCDs in runs (fh_device.hpp), in a launch of `tiles`: 16 KiB of input
// each, respectively 8 KiB of fp32 output.  The quantiser gains in fp32 from some 200 MB on: with runs of 128 a plan's 2 GiB both
// ways 868 -> 819 us, 1 GiB 398 -> 390, 240 MB of feature maps 89.5 -> 88.4; 278 MB 103.4 and 103.0, 60 MB 26.5 and 27.0; bf16 loses
// (encoder set 398 -> 407).  The restore of fp32 with runs of 64: encoder set 398 -> 379 us, 126 MB of it 41.0 -> 39.1, the plan
// 868 -> 854, MobileNetV2-style set 201 -> 197, 60 MB 26.5 and 26.3; runs of 32 gain a half of that, of 128 as much.  Restoring bf16 gains
// nothing (280 to 286 us), nor do the routed forms.  (A kernel of its own each: the test in the others cost a set of 60 MB 0.3 us of 25.6.)
inline bool compress_in_runs(uint32_t tiles) { return tiles >= 12288; }
inline bool restore_in_runs(uint32_t tiles) { return tiles >= 8192; }

// Whether the routed quantiser or its restore takes one tensor's descriptor in a short argument segment (fh_batch.hpp).  One tensor of
// 1.6 MB, both ways, 10.0 us with the batch's arguments and 8.5 with these, the whole chain on it 90.3 and 88.9.  Putting the
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

// Whether the count pass sets the mask as it adds to the counters, or a launch behind it does.  The additions are then waited for, and
// a wide tensor's workgroup has many: 3 tensors of 3072 channels 52 us with the launch and 56 without, 3 of 16384 128 and
// 154, 24 of 768 78 and 76, 18 of 1024 131 and 126, one of 768 17.9 and 16.9.
inline bool mask_with_the_counts(int64_t channels) { return channels <= 1024; }

// The Huffman encoder's group sums in a launch of `groups` altogether: scanned by a kernel between the count and the write
// pass, or every workgroup of the write pass adds up those before its own.  Adding up saves that launch and makes every
// workgroup of the write pass take longer, so what counts is how many of those there are.  Encoding, scanned and not: one
// stream of 64 groups 36.9 and 36.3 us, of 1024 76.4 and 73.7, of 4096 203.4 and 200.8, of 6000 317 and 317, of 12288
// 599 and 609; 24 streams of 335 groups 394.5 and 395.7, 24 of 1024 1108 and 1124, six of 4096 1122 and 1151.
inline bool group_sums_are_scanned(int64_t groups) { return groups > 4096; }

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
