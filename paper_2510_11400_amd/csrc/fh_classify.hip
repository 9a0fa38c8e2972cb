// Channel classification on gfx950: outliers by the k-sigma rule, counted per channel
// (paper Section 4.4.1: outliers are found with the empirical three-sigma rule and
// channels are sorted into salient and normal ones).  Contract and definition:
// include/fedhybrid.h.
//
// Two streaming passes over the tensor:
//   1. moments: pairwise binary64 sums of x and x*x.  The balanced tree of the
//      definition is walked in 1024-element spans (one per wave): inside a lane over its
//      consecutive elements, across the 64 lanes by xor 1, 2, 4, ... 32, across the rows of
//      the span, and then across spans by the same routine applied to the partial sums
//      (1024 partials per wave) until one pair is left.  Binary64 addition is commutative,
//      so a butterfly exchange forms exactly the tree's nodes; partial sums of different
//      rows and of the two moments are spread over the lanes (reduce-scatter) so that
//      each exchange level handles half of what the level before did.
//   2. count: d = (double)x - mean, outlier iff d*d > threshold; outliers are rare, so
//      each lane keeps a bit mask of its 16 elements and only set bits pay for the
//      channel index (division by invariant integers through multiply-high) and an LDS
//      histogram increment; the histogram is flushed with one global atomic per
//      non-zero bin and workgroup.  Where the workspace has room, the first pass leaves the
//      range of the values of every 128 elements behind, and this one reads only the pieces
//      whose range reaches beyond the threshold.
#include "../../include/fedhybrid.h"

#include "fh_batch.hpp"
#include "fh_channels.hpp"
#include "fh_stages.hpp"
#include "fh_device.hpp"
#include "fh_moments.hpp"
#include "fh_rules.hpp"

#include <limits.h>

#include <mutex>

namespace fh {
namespace {

constexpr int kThreads = 256;
constexpr int kWavesPerBlock = kThreads / kWave;
constexpr int kMaxChannels = 16384;

// ---- per-kernel descriptors (fh_batch.hpp: up to kBatch tensors per launch) ----------------
struct MomentsItem { const void* x; int64_t numel; f64x2* partial; uint32_t* ranges; Cleared cleared; };
struct ReduceItem  { const f64x2* in; int64_t count; f64x2* out; };
struct EmptyItem   { double* stats; Cleared cleared; };
struct MaskItem    { const uint32_t* counts; uint8_t* mask; int64_t min_outliers; int32_t channels; };

// ---- pass 1a: spans of the tensor ------------------------------------------------------
template <typename InT> struct Span;
template <> struct Span<float> {            // 4 rows of 256, 4 consecutive elements per lane
    static constexpr int ROWS = 4, EPL = 4;
    __device__ static __forceinline__ void widen(const u32x4& w, float (&x)[EPL]) {
        const f32x4 v = __builtin_bit_cast(f32x4, w);
        x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
    }
    __device__ static __forceinline__ float one(const float* p) { return *p; }
};
template <> struct Span<uint16_t> {         // 2 rows of 512, 8 consecutive elements per lane
    static constexpr int ROWS = 2, EPL = 8;
    __device__ static __forceinline__ void widen(const u32x4& v, float (&x)[EPL]) {
        x[0] = bf16_lo(v.x); x[1] = bf16_hi(v.x); x[2] = bf16_lo(v.y); x[3] = bf16_hi(v.y);
        x[4] = bf16_lo(v.z); x[5] = bf16_hi(v.z); x[6] = bf16_lo(v.w); x[7] = bf16_hi(v.w);
    }
    __device__ static __forceinline__ float one(const uint16_t* p) {
        return __builtin_bit_cast(float, (uint32_t)*p << 16);
    }
};

// ---- value ranges ------------------------------------------------------------------------
// Can a piece hold an outlier?  x -> (x - mean)^2 in binary64 rises on either side of the mean, rounding included, so
// its largest values over a range are at the range's ends.  (Ends that compare as NaN -- infinities or NaNs among the
// statistics -- count as "yes".)
__device__ __forceinline__ bool may_hold_outliers(uint32_t range, double mean, double threshold)
{
    const double low = (double)bf16_lo(range) - mean, high = (double)bf16_hi(range) - mean;
    return !(low * low <= threshold && high * high <= threshold);
}

// The reads are the time.  Two forms: up to kLargeLaunch bytes a wave takes one span and the tiles go to the workgroups
// in order.  A LARGE launch gives a wave 4 KiB (one span of fp32, two of bf16) and each XCD a contiguous eighth of the
// tiles: dealt out one by one, as the hardware does, the lines of partial sums and ranges are written from two L2s, and
// when the tensors come from HBM those few bytes cost as much as their lines travel.  First pass of a launch, one span in
// order against LARGE, us:  bf16 8 MB 4.0 / 4.9, 50 MB 11.1 / 11.3, 100 MB 20.4 / 20.0, 180 MB 35.1 / 31.8,
// 750 MB 137 / 121; fp32 40 MB 9.5 / 10.1, 134 MB 22.5 / 22.6, 557 MB 91 / 87.
constexpr int64_t kLargeLaunch = (int64_t)96 << 20;
__device__ __forceinline__ uint32_t tile_of_block()
{
    const uint32_t each = gridDim.x / kXcds;                  // the last gridDim.x mod 8 stay where they are
    return blockIdx.x < each * kXcds ? (blockIdx.x % kXcds) * each + blockIdx.x / kXcds : blockIdx.x;
}
template <typename InT, bool LARGE>
__device__ __forceinline__ void moments_of(const MomentsItem& it, const uint32_t block)
{
    constexpr int SPANS = LARGE ? 4 / Span<InT>::ROWS : 1, ROWS = SPANS * Span<InT>::ROWS, EPL = Span<InT>::EPL, ROW = kWave * EPL;
    const InT* x = static_cast<const InT*>(it.x);
    const int64_t numel = it.numel;
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t span = ((int64_t)block * kWavesPerBlock + wave) * SPANS;
    const int64_t base = span * kSpan;
    constexpr int64_t kOfBlock = (int64_t)kWavesPerBlock * SPANS * kSpan;
    clear_counters<kThreads>(it.cleared, block, (uint32_t)((numel + kOfBlock - 1) / kOfBlock));
    if (base >= numel) return;                                // wave-uniform
    const InT* xs = x + base;
    float v[ROWS][EPL];
    const bool interior = base + SPANS * kSpan <= numel;
    const auto whole_row = [&](int r) { return stream_load(reinterpret_cast<const u32x4*>(xs + (r * ROW + lane * EPL))); };
    const auto last_row = [&](int r) {
#pragma unroll
        for (int j = 0; j < EPL; ++j) {
            const uint32_t e = r * ROW + lane * EPL + j;
            v[r][j] = base + e < numel ? Span<InT>::one(xs + e) : 0.0f;
        }
    };
    if (LARGE && ROWS == Span<InT>::ROWS) {
        // Large launches of fp32 alone: with a test around every row the rows behind the first are requested once it is
        // there, and the classification of the 557 MiB set takes 108.5 us, not 109.4.
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            if (interior) Span<InT>::widen(whole_row(r), v[r]);
            else last_row(r);
        }
    } else if (interior) {                                    // one branch around all rows: none waits for another
        u32x4 w[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) w[r] = whole_row(r);
#pragma unroll
        for (int r = 0; r < ROWS; ++r) Span<InT>::widen(w[r], v[r]);
    } else {
#pragma unroll
        for (int r = 0; r < ROWS; ++r) last_row(r);
    }
    leave_moments<SPANS>(v, it.partial + span, it.ranges ? it.ranges + span * kPieces : nullptr,
                         (numel - base + kSpan - 1) / kSpan, lane);
}

template <typename InT, bool LARGE>
__global__ __launch_bounds__(kThreads) void moments_kernel(const Batch<MomentsItem> args)
{
    uint32_t block;
    const MomentsItem& it = args.item[batch_item(args, LARGE ? tile_of_block() : blockIdx.x, block)];
    moments_of<InT, LARGE>(it, block);
}
template <typename InT>
__global__ __launch_bounds__(kThreads) void moments_one_kernel(const MomentsItem it)
{
    moments_of<InT, false>(it, blockIdx.x);
}

// ---- pass 1b: spans of partial sums (4 rows of 256 pairs, 4 consecutive pairs per lane) --
template <typename Args>
__global__ __launch_bounds__(kThreads) void reduce_partials_kernel(const Args args)
{
    constexpr int ROWS = 4, EPL = 4, ROW = kWave * EPL;
    uint32_t block;
    const ReduceItem& it = item_of(args, blockIdx.x, block);
    const f64x2* in = it.in;
    const int64_t count = it.count;
    f64x2* out = it.out;
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t span = (int64_t)block * kWavesPerBlock + wave;
    const int64_t base = span * kSpan;
    if (base >= count) return;
    double a[ROWS], b[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        double d[EPL], q[EPL];
#pragma unroll
        for (int j = 0; j < EPL; ++j) {
            const int64_t i = base + r * ROW + lane * EPL + j;
            const f64x2 p = i < count ? in[i] : f64x2{0.0, 0.0};
            d[j] = p.x; q[j] = p.y;
        }
        a[r] = local_tree<EPL>(d);
        b[r] = local_tree<EPL>(q);
    }
    double s1, s2;
    both_moments(span_tree<1>(a, b, lane), lane, s1, s2);
    if (lane == 0) out[span] = f64x2{s1, s2};
}

// A tensor without elements: nothing else is launched for it.
struct EmptyBatch { EmptyItem item[kBatch]; };
__global__ __launch_bounds__(kThreads) void no_elements_kernel(const EmptyBatch args)
{
    const EmptyItem& it = args.item[blockIdx.x];
    clear_counters<kThreads>(it.cleared, 0u, 1u);
    if (threadIdx.x < 4) it.stats[threadIdx.x] = 0.0;
}

// ---- the last level of the tree (at most 1024 partial sums), then mean, variance and threshold -----------------
// The first wave of every workgroup of the count pass does this for itself, the first workgroup of a tensor writes it down: as
// a launch between the passes it was 4.7 us and the gap before it, here the other waves clear the histogram and the ranges are on
// their way meanwhile.  One tensor of 12 MB 16.9 -> 15.8 us, of 50 MB 29.7 -> 28.4, three of 50 MB 50.7 -> 48.4; on large sets the pass
// takes longer by as much as the launch took, and where its workgroups are short by more: there the launch is left (limits_apart, fh_rules.hpp).
struct LastLevel {
    const f64x2* in;                                          // the partial sums
    int32_t      count;
    double       k_sigma;
    double*      stats;
};
struct Limits { double mean, threshold; };
__device__ __forceinline__ Limits limits_of(const LastLevel& it, int64_t numel, uint32_t lane, bool write)      // one wave
{
    constexpr int ROWS = 4, EPL = 4, ROW = kWave * EPL;
    double a[ROWS], b[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        a[r] = b[r] = 0.0;
        if (r * ROW >= it.count) continue;                    // wave-uniform
        double d[EPL], q[EPL];
#pragma unroll
        for (int j = 0; j < EPL; ++j) {
            const int32_t i = r * ROW + (int32_t)lane * EPL + j;
            const f64x2 p = i < it.count ? it.in[i] : f64x2{0.0, 0.0};
            d[j] = p.x; q[j] = p.y;
        }
        a[r] = local_tree<EPL>(d);
        b[r] = local_tree<EPL>(q);
    }
    double s1, s2;
    both_moments(span_tree<1>(a, b, lane), lane, s1, s2);     // in every lane
    const double n = (double)numel;
    const double mean = (s1 + 0.0) / n;                       // a total of -0.0 counts as +0.0; IEEE division
    const double mean_sq = mean * mean;
    double variance = s2 / n - mean_sq;
    if (!(variance > 0.0)) variance = 0.0;
    const double threshold = (it.k_sigma * it.k_sigma) * variance;
    if (write && lane == 0) {
        it.stats[0] = mean;
        it.stats[1] = variance;
        it.stats[2] = threshold;
        it.stats[3] = n;
    }
    return Limits{mean, threshold};
}

// The same as a launch of its own, a wave for each tensor.
struct LimitsItem { LastLevel last; int64_t numel; };
struct LimitsBatch { LimitsItem item[kBatch]; };
__global__ __launch_bounds__(kWave) void limits_kernel(const LimitsBatch args)
{
    const LimitsItem& it = args.item[blockIdx.x];
    limits_of(it.last, it.numel, threadIdx.x, true);
}

// ---- pass 2: outliers per channel ----------------------------------------------------------
// Channel of an outlier: division by `inner` and `channels` through the small-dividend
// divider of fh_channels.hpp (dividends stay below divisor + 8 * 1024 here).
struct CountArgs {
    const void* x;
    int64_t numel;
    LastLevel last;
    uint32_t* counts;
    SmallDiv inner, channels;
    int32_t spans_per_wave;                                   // consecutive spans one wave walks
    const uint32_t* ranges;                                   // of the tensor's pieces (count_marked_kernel)
    uint8_t* mask;                                            // cleared; null: it is taken from the counts behind the pass
    int64_t min_outliers;
};

// A workgroup's histogram to the tensor's counters.  The additions to a counter follow one another, so just one of them takes it
// over the bound, and that one sets the mask: no launch behind the pass that reads the counters again (557 MiB set 108.5 -> 106.5
// us).  An addition whose result is waited for costs more than one that is not, so that is for tensors of few channels and
// launches that are not too large (fh_rules.hpp).
template <int THREADS>
__device__ __forceinline__ void add_outliers(const CountArgs& args, const uint32_t* hist)
{
    const uint32_t channels = args.channels.d;
    uint32_t* const counts = args.counts;
    uint8_t* const mask = args.mask;
    const int64_t bound = args.min_outliers;
    if (!mask) {                                              // workgroup-uniform
        for (uint32_t c = threadIdx.x; c < channels; c += THREADS) {
            const uint32_t v = hist[c];
            if (v) atomicAdd(&counts[c], v);
        }
        return;
    }
    for (uint32_t c = threadIdx.x; c < channels; c += THREADS) {
        const uint32_t v = hist[c];
        if (!v) continue;
        const uint32_t before = atomicAdd(&counts[c], v);
        if ((int64_t)before < bound && (int64_t)before + v >= bound) mask[c] = 1;
    }
}

__device__ __forceinline__ double uniform(double v)            // the same in all lanes, into scalar registers
{
    const u32x2 w = __builtin_bit_cast(u32x2, v);
    const uint32_t low = w.x, high = w.y;
    return __builtin_bit_cast(double, ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)high) << 32) |
                                          (uint32_t)__builtin_amdgcn_readfirstlane((int)low));
}

// AHEAD: a launch in which some wave walks more than one span.  APART: the limits are there (limits_apart, fh_rules.hpp).
constexpr int kAhead = 3;                         // spans requested before the one that is looked at
template <typename InT, bool AHEAD, bool APART, typename Args>
__global__ __launch_bounds__(kThreads) void count_outliers_kernel(const Args batch)
{
    constexpr int ROWS = Span<InT>::ROWS, EPL = Span<InT>::EPL, ROW = kWave * EPL;
    extern __shared__ uint32_t hist[];
    __shared__ Limits limits;
    uint32_t block;
    const CountArgs& args = item_of(batch, blockIdx.x, block);
    const uint32_t C = args.channels.d;
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (!APART && wave == 0) {
        const Limits found = limits_of(args.last, args.numel, lane, block == 0);
        if (lane == 0) limits = found;
    }
    for (uint32_t c = threadIdx.x; c < C; c += kThreads) hist[c] = 0u;
    __syncthreads();
    const double mean = APART ? args.last.stats[0] : uniform(limits.mean), threshold = APART ? args.last.stats[2] : uniform(limits.threshold);
    const InT* x = static_cast<const InT*>(args.x);
    const int64_t numel = args.numel;
    // this wave's spans: first_span, first_span + 1, ...
    const int64_t first_span = ((int64_t)block * kWavesPerBlock + wave) * args.spans_per_wave;
    int64_t base = first_span * kSpan;
    // position of the span's first element: rem = index inside the channel run, chan = channel
    uint32_t rem = 0, chan = 0;
    if (base < numel) {
        const uint64_t run = (uint64_t)base / args.inner.d;   // once per wave
        rem = (uint32_t)((uint64_t)base - run * args.inner.d);
        chan = (uint32_t)(run % C);
    }
    // The rows of the spans ahead are requested before this one's are looked at: a wave walks its spans one after
    // the other, and with one span in flight per wave the device does not hold enough bytes in flight to cover the
    // memory latency (measured on bf16 [tokens][hidden] tensors with 6 to 16 spans per wave: 32 -> 28 us per 80 MB
    // with one span ahead; a single such tensor is 1.5 waves per SIMD, and with three spans ahead its pass takes
    // as long as the first pass over it).  The ring of kAhead + 1 spans has constant indices: the walk is
    // unrolled by that many.
    constexpr int RING = AHEAD ? kAhead + 1 : 1;
    u32x4 ring[RING][ROWS];
    const auto request = [&](int64_t at, u32x4 (&w)[ROWS]) {  // whole spans only: the last one of a tensor is read element by element
        if (at + kSpan <= numel) {
#pragma unroll
            for (int r = 0; r < ROWS; ++r) w[r] = stream_load(reinterpret_cast<const u32x4*>(x + at + r * ROW + lane * EPL));
        }
    };
    const int spans = args.spans_per_wave;
    if (AHEAD) {
#pragma unroll
        for (int k = 0; k < kAhead; ++k)
            if (k < spans && base + (int64_t)k * kSpan < numel) request(base + (int64_t)k * kSpan, ring[k]);
    }
    // one span: the outliers of its rows into the histogram, then (rem, chan) and base move on by a span
    const auto look = [&](const u32x4 (&now)[ROWS], bool interior) {
        const InT* xs = x + base;
        uint32_t bits = 0u;                                   // bit r * EPL + j: that element is an outlier
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            float v[EPL];
            const uint32_t e0 = r * ROW + lane * EPL;
            if (interior) {
                Span<InT>::widen(now[r], v);
            } else {
#pragma unroll
                for (int j = 0; j < EPL; ++j)
                    v[j] = (base + e0 + j < numel) ? Span<InT>::one(xs + e0 + j) : __builtin_bit_cast(float, 0x7fc00000u);
            }
#pragma unroll
            for (int j = 0; j < EPL; ++j) {
                const double d = (double)v[j] - mean;
                if (d * d > threshold) bits |= 1u << (r * EPL + j);          // false for the NaN filler
            }
        }
        while (bits) {                                        // rare: about k-sigma tail mass * 16 per lane
            const uint32_t k2 = (uint32_t)__builtin_ctz(bits);
            bits &= bits - 1u;
            const uint32_t off = (k2 / EPL) * ROW + lane * EPL + (k2 % EPL);   // element offset inside the span
            const uint32_t runs = div_small(rem + off, args.inner);           // channel runs crossed from `chan`
            const uint32_t cc = chan + runs;
            const uint32_t c = cc - div_small(cc, args.channels) * C;
            atomicAdd(&hist[c], 1u);
        }
        const uint32_t t = rem + kSpan;
        const uint32_t runs = div_small(t, args.inner);
        rem = t - runs * args.inner.d;
        const uint32_t cc = chan + runs;
        chan = cc - div_small(cc, args.channels) * C;
        base += kSpan;
    };
    for (int s0 = 0; s0 < spans && base < numel; s0 += RING) {
        // A round whose spans, and the spans requested during it, are all whole and all this wave's runs without
        // a test around any load: only then can the waits be for the oldest request alone and not for all of them.
        if (AHEAD && s0 + RING + kAhead <= spans && base + (int64_t)(RING + kAhead) * kSpan <= numel) {
#pragma unroll
            for (int k = 0; k < RING; ++k) {
                u32x4 (&ahead)[ROWS] = ring[(k + kAhead) % RING];
#pragma unroll
                for (int r = 0; r < ROWS; ++r)
                    ahead[r] = stream_load(reinterpret_cast<const u32x4*>(x + base + (int64_t)kAhead * kSpan + r * ROW + lane * EPL));
                look(ring[k], true);
            }
            continue;
        }
#pragma unroll
        for (int k = 0; k < RING; ++k) {
            const int s = s0 + k;
            if (s >= spans || base >= numel) break;
            if (AHEAD && s + kAhead < spans && base + (int64_t)kAhead * kSpan < numel)
                request(base + (int64_t)kAhead * kSpan, ring[(k + kAhead) % RING]);
            if (!AHEAD) request(base, ring[k]);
            look(ring[k], base + kSpan <= numel);
        }
    }
    __syncthreads();
    add_outliers<kThreads>(args, hist);
}

// The same where the first pass left ranges behind.  A wave looks at the ranges of eight spans at once, a lane per
// piece, lists the pieces that may hold an outlier, and reads those: eight lanes to a piece, a lane's elements the
// ones it would have in a span walked whole.  Two rounds of eight pieces are requested together: with four the kernel
// takes 112 vector registers in fp32 and four waves fit a SIMD, with two 82 (64 in bf16).  What bounds the
// pass is what the data leave to read: nothing but the salient channels' share on feature maps with outliers
// clustered in channels (557 MiB set: 15 us, the kernel above 95), a quarter to a third of the lines of
// [tokens][hidden] tensors (Gaussian tails alone put an outlier in 3 of 10 pieces; 720 MiB of bf16: 114 us against 160,
// with clustered outliers 53 against 154).  With an outlier in most pieces it reads nearly all of the tensor, in as many
// waves as the rules of fh_rules.hpp give the launch: 23 us for 100 MB of fp32 with 3072 channels, the kernel above 25.
constexpr int kLook = 8;                          // spans whose ranges a wave looks at together: 64 pieces
constexpr int kRounds = 2;                        // rounds of eight pieces requested together
template <typename InT, int WAVES, bool APART, typename Args>
__global__ __launch_bounds__(WAVES * kWave) void count_marked_kernel(const Args batch)
{
    constexpr int kThreads = WAVES * kWave;
    constexpr int ROWS = Span<InT>::ROWS, EPL = Span<InT>::EPL, ROW = kWave * EPL;
    extern __shared__ uint32_t hist[];
    __shared__ Limits limits;
    uint32_t block;
    const CountArgs& args = item_of(batch, blockIdx.x, block);
    const uint32_t C = args.channels.d;
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const InT* x = static_cast<const InT*>(args.x);
    const int64_t numel = args.numel, all_spans = (numel + kSpan - 1) / kSpan;
    const int64_t first = ((int64_t)block * WAVES + wave) * args.spans_per_wave;
    const int64_t stop = first + args.spans_per_wave < all_spans ? first + args.spans_per_wave : all_spans;
    const auto range_of = [&](int64_t span) { return span + (lane >> 3) < stop ? args.ranges[span * kPieces + lane] : 0u; };
    uint32_t range = range_of(first);                         // in flight while the counters are cleared
    if (!APART && wave == 0) {
        const Limits found = limits_of(args.last, numel, lane, block == 0);
        if (lane == 0) limits = found;
    }
    for (uint32_t c = threadIdx.x; c < C; c += kThreads) hist[c] = 0u;
    __syncthreads();
    const double mean = APART ? args.last.stats[0] : uniform(limits.mean), threshold = APART ? args.last.stats[2] : uniform(limits.threshold);
    for (int64_t span0 = first; span0 < stop; span0 += kLook) {          // wave-uniform
        const bool mark = span0 + (lane >> 3) < stop && may_hold_outliers(range, mean, threshold);
        const uint64_t marks = __ballot(mark);
        if (span0 + kLook < stop) range = range_of(span0 + kLook);
        const uint32_t pieces = (uint32_t)__popcll(marks);
        if (pieces == 0u) continue;
        // lane k of `list`: the k-th marked piece (the unmarked ones behind them, so that every lane sends and receives)
        const uint32_t before = __builtin_amdgcn_mbcnt_hi((uint32_t)(marks >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)marks, 0u));
        const int list = __builtin_amdgcn_ds_permute((int)((mark ? before : pieces + lane - before) << 2), (int)lane);
        // position of the first span's first element: rem = index inside the channel run, chan = channel
        const int64_t base = span0 * kSpan;
        const uint64_t run = (uint64_t)base / args.inner.d;
        const uint32_t rem = (uint32_t)((uint64_t)base - run * args.inner.d), chan = (uint32_t)(run % C);
        const int64_t whole = (numel - base) / kSpan;         // spans from here on that are whole
        for (uint32_t p0 = 0; p0 < pieces; p0 += 8u * kRounds) {
            uint32_t at[kRounds];                             // the lane's first element, from the first span's; ~0: no piece
            bool inside[kRounds];                             // all of the piece's span exists
            u32x4 w[kRounds][ROWS];
#pragma unroll
            for (int k = 0; k < kRounds; ++k) {
                const uint32_t p = p0 + 8u * k + (lane >> 3);            // at most 63
                const uint32_t piece = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(p << 2), list);
                inside[k] = p < pieces && (int64_t)(piece >> 3) < whole;
                at[k] = p < pieces ? (piece >> 3) * (uint32_t)kSpan + ((piece & 7u) * 8u + (lane & 7u)) * EPL : ~0u;
                if (inside[k]) {
#pragma unroll
                    for (int r = 0; r < ROWS; ++r) w[k][r] = stream_load(reinterpret_cast<const u32x4*>(x + base + at[k] + r * ROW));
                }
            }
#pragma unroll
            for (int k = 0; k < kRounds; ++k) {
                if (p0 + 8u * k >= pieces) break;             // wave-uniform
                if (at[k] == ~0u) continue;
                uint32_t bits = 0u;                           // bit r * EPL + j: that element is an outlier
#pragma unroll
                for (int r = 0; r < ROWS; ++r) {
                    float v[EPL];
                    if (inside[k]) {
                        Span<InT>::widen(w[k][r], v);
                    } else {
#pragma unroll
                        for (int j = 0; j < EPL; ++j) {
                            const int64_t i = base + at[k] + r * ROW + j;
                            v[j] = i < numel ? Span<InT>::one(x + i) : __builtin_bit_cast(float, 0x7fc00000u);
                        }
                    }
#pragma unroll
                    for (int j = 0; j < EPL; ++j) {
                        const double d = (double)v[j] - mean;
                        if (d * d > threshold) bits |= 1u << (r * EPL + j);          // false for the NaN filler
                    }
                }
                while (bits) {
                    const uint32_t k2 = (uint32_t)__builtin_ctz(bits);
                    bits &= bits - 1u;
                    const uint32_t off = at[k] + (k2 / EPL) * ROW + (k2 % EPL);       // below 8 * 1024
                    const uint32_t cc = chan + div_small(rem + off, args.inner);      // channel runs crossed from `chan`
                    atomicAdd(&hist[cc - div_small(cc, args.channels) * C], 1u);
                }
            }
        }
    }
    __syncthreads();
    add_outliers<kThreads>(args, hist);
}

template <typename Args>
__global__ __launch_bounds__(kThreads) void mask_kernel(const Args args)
{
    uint32_t block;
    const MaskItem& it = item_of(args, blockIdx.x, block);
    const int c = block * kThreads + threadIdx.x;
    if (c < it.channels) it.mask[c] = (int64_t)it.counts[c] >= it.min_outliers ? 1 : 0;
}

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

}  // namespace
}  // namespace fh

extern "C" {

size_t fh_classify_workspace_bytes(int64_t numel)
{
    // one {sum x, sum x*x} pair per 1024-element span, then per 1024 of those, ... down to one
    if (numel <= 0) return 16;
    size_t pairs = 0;
    int64_t m = fh::ceil_div(numel, fh::kSpan);
    for (;;) {
        pairs += (size_t)m;
        if (m == 1) break;
        m = fh::ceil_div(m, fh::kSpan);
    }
    return pairs * 16;
}

size_t fh_classify_workspace_bytes_ranges(int64_t numel)
{
    return fh_classify_workspace_bytes(numel) + fh::range_bytes(numel);
}

}  // extern "C"

// ---- partial sums in a buffer of the library's own -------------------------------------------
// For callers that cannot allocate (HIP graph capture, serving loops, harnesses that forbid it):
// the workspace of the partial-sum tree as a device array that is part of the code object.  Each
// GPU the library runs on holds its own copy at its own address until the process ends; every
// call on a GPU shares it, so calls that overlap on one GPU race.  Nothing in it has to start
// at zero: every level of the tree is written in full before it is read.
constexpr size_t kScratchBytes = (size_t)4 << 20;           // serves up to 2^28 - 2^18 elements
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {

using namespace fh;

// The device address of `scratch` on the current device.  In host code the array's name is only
// a handle for hipGetSymbolAddress, never an address a kernel may be given; the address is
// asked for once per device, with that device current, and kept.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_lock;
void* g_scratch_ptr[kMaxDevices] = {};

fh_status scratch_of_current_device(void** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return FH_ERR_LAUNCH;
    std::lock_guard<std::mutex> hold(g_scratch_lock);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return FH_ERR_LAUNCH;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return FH_OK;
}

fh_status check_item(const fh_classify_item& it, int64_t* numel_out)
{
    if (it.x_dtype != FH_F32 && it.x_dtype != FH_BF16) return FH_ERR_BAD_DTYPE;
    if (it.reserved != 0) return FH_ERR_BAD_PARAM;
    if (it.outer < 0 || it.inner < 1 || it.channels < 1 || it.channels > kMaxChannels) return FH_ERR_BAD_SHAPE;
    if (it.inner > (int64_t)1 << 31 || it.outer > (int64_t)1 << 40) return FH_ERR_BAD_SHAPE;
    if (!(it.k_sigma > 0.0) || it.min_outliers < 1) return FH_ERR_BAD_PARAM;
    const double total = (double)it.outer * (double)it.channels * (double)it.inner;
    if (total > (double)((int64_t)1 << 40)) return FH_ERR_BAD_NUMEL;
    const int64_t numel = it.outer * it.channels * it.inner;
    if (!it.workspace || !it.stats || !it.counts || !it.mask || (numel > 0 && !it.x)) return FH_ERR_NULL;
    auto misaligned = [](const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) != 0; };
    if (misaligned(it.x, 16) || misaligned(it.workspace, 16) || misaligned(it.stats, 8) || misaligned(it.counts, 4))
        return FH_ERR_ALIGNMENT;
    if (it.workspace_cap < fh_classify_workspace_bytes(numel)) return FH_ERR_BUFFER_TOO_SMALL;
    *numel_out = numel;
    return FH_OK;
}

// One run of up to kBatch tensors of one dtype: two to five launches, each covering all of them.  The tensors either all
// have a place for their ranges or all have none.
fh_status run_classify(const fh_classify_item* items, uint32_t* const* ranges, const int64_t* numels, int n, bool masks,
                       bool first_pass_done, hipStream_t s)
{
    const bool marked = ranges[0] != nullptr;
    const dim3 block(kThreads);
    const int dtype = items[0].x_dtype;
    int64_t elements = 0, spans = 0;                          // of the launch
    for (int i = 0; i < n; ++i) {
        elements += numels[i];
        spans += ceil_div(numels[i], kSpan);
    }
    const bool large = elements * (dtype == FH_F32 ? 4 : 2) > kLargeLaunch;
    f64x2* level[kBatch];
    int64_t m[kBatch];
    const int64_t per_block = kWavesPerBlock * (dtype == FH_F32 || !large ? 1 : 2);      // spans of a workgroup of the first pass

    Batch<MomentsItem> mb;
    reset(mb);
    for (int i = 0; i < n; ++i) {
        level[i] = static_cast<f64x2*>(items[i].workspace);
        m[i] = numels[i] > 0 ? ceil_div(numels[i], kSpan) : 0;
        if (numels[i] > 0 && !first_pass_done && !push(mb, MomentsItem{items[i].x, numels[i], level[i], ranges[i], cleared_of(items[i])}, ceil_div(m[i], per_block)))
            return FH_ERR_BAD_NUMEL;
    }
    if (mb.count > 0) {
        seal(mb);
        const dim3 grid(mb.block_start[mb.count]);
        if (mb.count == 1 && !large) {                        // (a large launch needs its grid's size)
            static_assert(sizeof(MomentsItem) <= kOneLaunchArgs, "the descriptor of one tensor is a short argument segment");
            if (dtype == FH_F32) hipLaunchKernelGGL((moments_one_kernel<float>), grid, block, 0, s, mb.item[0]);
            else hipLaunchKernelGGL((moments_one_kernel<uint16_t>), grid, block, 0, s, mb.item[0]);
        } else if (dtype == FH_F32) {
            if (large) hipLaunchKernelGGL((moments_kernel<float, true>), grid, block, 0, s, mb);
            else hipLaunchKernelGGL((moments_kernel<float, false>), grid, block, 0, s, mb);
        } else {
            if (large) hipLaunchKernelGGL((moments_kernel<uint16_t, true>), grid, block, 0, s, mb);
            else hipLaunchKernelGGL((moments_kernel<uint16_t, false>), grid, block, 0, s, mb);
        }
    }
    for (;;) {                                                // tree levels above the first, where needed
        Batch<ReduceItem> rb;
        reset(rb);
        for (int i = 0; i < n; ++i) {
            if (m[i] <= kSpan) continue;                      // the last <= 1024 partials are the count pass's
            const int64_t next = ceil_div(m[i], kSpan);
            f64x2* out = level[i] + m[i];
            push(rb, ReduceItem{level[i], m[i], out}, ceil_div(next, kWavesPerBlock));
            level[i] = out;
            m[i] = next;
        }
        if (rb.count == 0) break;
        seal(rb);
        const dim3 grid(rb.block_start[rb.count]);
        with_arguments(rb, [&](const auto& args) { hipLaunchKernelGGL((reduce_partials_kernel<FH_ARGS>), grid, block, 0, s, args); });
    }
    EmptyBatch eb;
    int empty = 0;
    for (int i = 0; i < n; ++i)
        if (numels[i] == 0) eb.item[empty++] = EmptyItem{static_cast<double*>(items[i].stats), cleared_of(items[i])};
    if (empty > 0) {
        for (int i = empty; i < kBatch; ++i) eb.item[i] = eb.item[0];
        hipLaunchKernelGGL(no_elements_kernel, dim3(empty), block, 0, s, eb);
    }

    Batch<CountArgs> cb;
    Batch<MaskItem> kb;
    reset(cb);
    reset(kb);
    int of_item[kBatch];                                      // the count pass's tensors among `items`
    int64_t widest = 0;
    for (int i = 0; i < n; ++i)
        if (numels[i] > 0 && items[i].channels > widest) widest = items[i].channels;
    const size_t lds = (size_t)widest * sizeof(uint32_t);
    const int waves = marked ? marked_waves_per_workgroup(widest) : kWavesPerBlock;
    for (int i = 0; i < n; ++i) {
        if (numels[i] == 0) continue;                         // no outliers: the cleared mask stands
        CountArgs a;
        a.x = items[i].x;
        a.numel = numels[i];
        a.last = LastLevel{level[i], (int32_t)m[i], items[i].k_sigma, static_cast<double*>(items[i].stats)};
        a.counts = static_cast<uint32_t*>(items[i].counts);
        a.inner = make_small_div((uint32_t)items[i].inner);
        a.channels = make_small_div((uint32_t)items[i].channels);
        // a workgroup clears `channels` histogram bins and adds the non-zero ones to the tensor's counters with
        // atomics that meet those of every other workgroup on a few cache lines: give it enough elements to make
        // that cheap, but no more (short workgroups measured faster on feature maps; 128 elements per bin and
        // wave on [tokens][hidden] tensors, where the outliers of ordinary activations touch most bins)
        const int64_t ch = items[i].channels;
        a.spans_per_wave = marked ? marked_spans_per_wave(spans, ceil_div(numels[i], kSpan), ch, widest)
                                  : (int32_t)(ch <= 512 ? 1 : ch / 128 < 16 ? ch / 128 : 16);
        a.ranges = ranges[i];
        if (marked) a.spans_per_wave *= marked_looks_per_wave(spans, ch);
        a.mask = nullptr;
        a.min_outliers = items[i].min_outliers;
        const int64_t per_block = (int64_t)a.spans_per_wave * waves * kSpan;
        of_item[cb.count] = i;
        if (!push(cb, a, ceil_div(numels[i], per_block))) return FH_ERR_BAD_NUMEL;
    }
    if (cb.count > 0) {
        seal(cb);
        const dim3 grid(cb.block_start[cb.count]);
        uint32_t of_one_span = 0;
        bool crowded = false;
        for (int k = 0; k < cb.count; ++k)
            if (cb.item[k].spans_per_wave == 1) {
                const uint32_t workgroups = cb.block_start[k + 1] - cb.block_start[k];
                of_one_span += workgroups;
                crowded = crowded || counters_are_crowded(workgroups, cb.item[k].channels.d);
            }
        const bool apart = limits_apart(marked, cb.count, grid.x, of_one_span, crowded);
        if (apart) {
            LimitsBatch lb;
            for (int k = 0; k < kBatch; ++k) {
                const CountArgs& a = cb.item[k < cb.count ? k : 0];
                lb.item[k] = LimitsItem{a.last, a.numel};
            }
            hipLaunchKernelGGL(limits_kernel, dim3(cb.count), dim3(kWave), 0, s, lb);
        }
        for (int k = 0; k < cb.count && masks; ++k) {
            const fh_classify_item& it = items[of_item[k]];
            // (counters of channels with 2^32 elements and more may wrap: the masks are then what they end at)
            const bool here = apart    ? mask_with_the_counts_apart(it.channels, marked, cb.count)
                              : marked ? mask_with_the_counts(it.channels)
                                       : mask_with_the_counts_unranged(it.channels, ceil_div(cb.item[k].numel, kSpan));
            if (here && it.outer * it.inner <= (int64_t)UINT32_MAX)
                cb.item[k].mask = static_cast<uint8_t*>(it.mask);
            else
                push(kb, MaskItem{cb.item[k].counts, static_cast<uint8_t*>(it.mask), it.min_outliers, (int32_t)it.channels},
                     ceil_div(it.channels, kThreads));
        }
        seal(kb);
        bool ahead = false;
        for (int k = 0; k < cb.count; ++k) ahead = ahead || cb.item[k].spans_per_wave > 1;
        const dim3 threads(marked ? waves * kWave : kThreads);
        if (apart && marked) {
            if (dtype == FH_F32) {
                if (waves == 4) hipLaunchKernelGGL((count_marked_kernel<float, 4, true, Batch<CountArgs>>), grid, threads, lds, s, cb);
                else hipLaunchKernelGGL((count_marked_kernel<float, 8, true, Batch<CountArgs>>), grid, threads, lds, s, cb);
            } else {
                if (waves == 4) hipLaunchKernelGGL((count_marked_kernel<uint16_t, 4, true, Batch<CountArgs>>), grid, threads, lds, s, cb);
                else hipLaunchKernelGGL((count_marked_kernel<uint16_t, 8, true, Batch<CountArgs>>), grid, threads, lds, s, cb);
            }
        } else if (apart) {
            if (dtype == FH_F32) {
                if (ahead) hipLaunchKernelGGL((count_outliers_kernel<float, true, true, Batch<CountArgs>>), grid, threads, lds, s, cb);
                else hipLaunchKernelGGL((count_outliers_kernel<float, false, true, Batch<CountArgs>>), grid, threads, lds, s, cb);
            } else {
                if (ahead) hipLaunchKernelGGL((count_outliers_kernel<uint16_t, true, true, Batch<CountArgs>>), grid, threads, lds, s, cb);
                else hipLaunchKernelGGL((count_outliers_kernel<uint16_t, false, true, Batch<CountArgs>>), grid, threads, lds, s, cb);
            }
        } else with_arguments(cb, [&](const auto& args) {
            if (marked && dtype == FH_F32) {
                if (waves == 4) hipLaunchKernelGGL((count_marked_kernel<float, 4, false, FH_ARGS>), grid, threads, lds, s, args);
                else hipLaunchKernelGGL((count_marked_kernel<float, 8, false, FH_ARGS>), grid, threads, lds, s, args);
            } else if (marked) {
                if (waves == 4) hipLaunchKernelGGL((count_marked_kernel<uint16_t, 4, false, FH_ARGS>), grid, threads, lds, s, args);
                else hipLaunchKernelGGL((count_marked_kernel<uint16_t, 8, false, FH_ARGS>), grid, threads, lds, s, args);
            } else if (dtype == FH_F32) {
                if (ahead) hipLaunchKernelGGL((count_outliers_kernel<float, true, false, FH_ARGS>), grid, threads, lds, s, args);
                else hipLaunchKernelGGL((count_outliers_kernel<float, false, false, FH_ARGS>), grid, threads, lds, s, args);
            } else {
                if (ahead) hipLaunchKernelGGL((count_outliers_kernel<uint16_t, true, false, FH_ARGS>), grid, threads, lds, s, args);
                else hipLaunchKernelGGL((count_outliers_kernel<uint16_t, false, false, FH_ARGS>), grid, threads, lds, s, args);
            }
        });
        if (kb.count > 0) {
            const dim3 of_masks(kb.block_start[kb.count]);
            with_arguments(kb, [&](const auto& args) { hipLaunchKernelGGL((mask_kernel<FH_ARGS>), of_masks, block, 0, s, args); });
        }
    }
    return hipGetLastError() == hipSuccess ? FH_OK : FH_ERR_LAUNCH;
}

// All tensors (checked): runs of one dtype that have ranges or have none, at most kBatch long.
// range_of(i, numel): where the ranges of tensor i go, or null.
template <typename RangeOf>
fh_status run_all(const fh_classify_item* items, int32_t count, bool masks, bool first_pass_done, hipStream_t s, RangeOf range_of)
{
    const auto numel_of = [items](int32_t i) { return items[i].outer * items[i].channels * items[i].inner; };
    int32_t i = 0;
    while (i < count) {
        int64_t numels[kBatch];
        uint32_t* ranges[kBatch];
        int n = 0;
        for (; i + n < count && n < kBatch && items[i + n].x_dtype == items[i].x_dtype; ++n) {
            numels[n] = numel_of(i + n);
            ranges[n] = range_of(i + n, numels[n]);
            if (!ranges[n] != !ranges[0]) break;
        }
        const fh_status st = run_classify(items + i, ranges, numels, n, masks, first_pass_done, s);
        if (st != FH_OK) return st;
        i += n;
    }
    return FH_OK;
}

}  // namespace

fh_status fh::classify_counts(const fh_classify_item* items, uint32_t* const* ranges, int32_t count, bool first_pass_done,
                              hipStream_t s)
{
    return run_all(items, count, false, first_pass_done, s, [ranges](int32_t i, int64_t) { return ranges[i]; });
}

extern "C" {

int32_t fh_classify_batch_capacity(void) { return fh::kBatchStated; }

fh_status fh_classify_channels_batch(const fh_classify_item* items, int32_t count, void* stream)
{
    if (count < 0) return FH_ERR_BAD_COUNT;
    if (count > 0 && !items) return FH_ERR_NULL;
    // all items are checked before the first launch
    for (int32_t i = 0; i < count; ++i) {
        int64_t numel;
        const fh_status st = check_item(items[i], &numel);
        if (st != FH_OK) return st;
    }
    // the ranges lie behind the partial sums, where there is room for them
    return run_all(items, count, true, false, static_cast<hipStream_t>(stream), [items](int32_t i, int64_t numel) -> uint32_t* {
        const size_t pairs = fh_classify_workspace_bytes(numel);
        if (items[i].workspace_cap < pairs + range_bytes(numel)) return nullptr;
        return reinterpret_cast<uint32_t*>(static_cast<unsigned char*>(items[i].workspace) + pairs);
    });
}

fh_status fh_classify_channels(const void* x, fh_dtype x_dtype, int64_t outer, int64_t channels, int64_t inner,
                               double k_sigma, int64_t min_outliers,
                               void* workspace, size_t workspace_cap,
                               void* stats, void* counts, void* mask, void* stream)
{
    fh_classify_item it;
    it.x = x; it.x_dtype = x_dtype; it.reserved = 0;
    it.outer = outer; it.channels = channels; it.inner = inner;
    it.k_sigma = k_sigma; it.min_outliers = min_outliers;
    it.workspace = workspace; it.workspace_cap = workspace_cap;
    it.stats = stats; it.counts = counts; it.mask = mask;
    return fh_classify_channels_batch(&it, 1, stream);
}

size_t fh_classify_static_scratch_bytes(void) { return kScratchBytes; }

fh_status fh_classify_channels_static(const void* x, fh_dtype x_dtype, int64_t outer, int64_t channels, int64_t inner,
                                      double k_sigma, int64_t min_outliers,
                                      void* stats, void* counts, void* mask, void* stream)
{
    // the size check comes first: a tensor the static buffer cannot serve is refused before
    // anything else is looked at, and before the buffer's address is asked for
    if (outer >= 0 && channels >= 1 && inner >= 1) {
        const double total = (double)outer * (double)channels * (double)inner;
        if (total > (double)((int64_t)1 << 40)) return FH_ERR_BAD_NUMEL;
        if (fh_classify_workspace_bytes(outer * channels * inner) > kScratchBytes) return FH_ERR_SCRATCH_LIMIT;
    }
    void* ws = nullptr;
    const fh_status st = scratch_of_current_device(&ws);
    if (st != FH_OK) return st;
    return fh_classify_channels(x, x_dtype, outer, channels, inner, k_sigma, min_outliers, ws, kScratchBytes,
                                stats, counts, mask, stream);
}

}  // extern "C"
