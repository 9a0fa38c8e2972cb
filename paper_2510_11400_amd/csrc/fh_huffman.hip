// Huffman coding of a byte stream on gfx950 (paper Section 4.4.1: the quantisation codes of
// the predictive form are encoded with Huffman coding; restoring starts with Huffman
// decoding).  The paper names the coder only; the definition used (tie-breaks, 24-bit limit,
// canonical codes, layout) is the one in include/fedhybrid.h.
//
// A variable-length code is sequential per symbol, so the stream is cut into chunks of 256
// symbols that start on a 32-bit word; the decoder gives a chunk to a thread, the encoder to
// sixteen lanes.  Encoding is stream compaction again:
//   histogram   LDS counters, one copy per bank and the copies interleaved, so that no two lanes
//               of a half-wave meet in a bank whatever the bytes are; added to the global
//               histogram at the end;
//   code        one workgroup: the used symbols are ranked by (count, symbol) in parallel, one
//               wave runs the two-queue construction over the ranked leaves (at most 255
//               merges, those that do not depend on each other side by side) and every leaf
//               walks up the tree for its depth; counts are halved and the construction
//               repeated while a code would exceed 24 bits; canonical codes;
//   count       a wave reads four chunks at a time with one 16-byte load per lane and adds the
//               code lengths up over each chunk's sixteen lanes: the chunk's length in words;
//   scan        the sums of groups of 256 chunks (a workgroup of the count pass) are scanned by
//               one workgroup, in launches of many groups; in others every workgroup of the
//               write pass adds up the sums before its own;
//   write       word counts become offsets (group base + a scan over the workgroup); a wave
//               then codes four chunks at a time, every lane placing the bits of its sixteen
//               symbols in an LDS area by OR, and stores the four chunks' words -- one
//               contiguous piece -- with consecutive lanes on consecutive words.
// Decoding needs no pass but one: the offsets are part of the stream.  A workgroup has the whole LDS of a compute unit.
// While the payload slice of up to 1024 chunks is on its way there it rebuilds the canonical tables from the 256 lengths
// (a lookup table, coarser for the short codes than for the longer; comparisons for the longest), and a thread decodes
// its chunk from LDS; the table serves several such groups in long streams.
// Everything here is integer work; results do not depend on launch geometry.
#include "../../include/fedhybrid.h"

#include "fh_batch.hpp"
#include "fh_rules.hpp"
#include "fh_scan.hpp"
#include "fh_stages.hpp"

namespace fh {
namespace {

constexpr int kChunk = 256;                        // symbols per chunk (= per thread)
constexpr int kThreads = 256;                      // of the passes that have a thread per symbol or per group
constexpr int kMaxLen = 24;
constexpr int kChunkWordsMax = kChunk * kMaxLen / 32;
constexpr int kHistCopies = 32;                     // one per LDS bank
constexpr int kHistThreads = 1024;
static_assert(kHistThreads * 16 == kHistRound, "a vector of sixteen symbols for each thread (fh_rules.hpp)");
// decode: 16-byte output vectors held back and stored together; 51 MB of index streams one at a time 54.5 us, 2 44.5, 4 44.4,
// with 8 the code no longer fits the instruction cache and takes 58.2
constexpr int kBurst = 4;
// decode: threads per workgroup, one workgroup per compute unit.  The payload slice in LDS is what limits the chunks in
// flight on a unit.  With 1024 threads the stage holds 768 chunks at 46 words (5.75 bits per symbol) and 1024 at 34.5: a
// stream whose chunks come to slightly more than 768 per unit (51 MB of index streams: 788) takes one pass and not two;
// four waves per SIMD then keep the LDS busy (44.4 us).  A launch of fewer chunks has 512 threads, half as many waves to a SIMD, and
// a stage of 61 words for each: 13 MB of index streams 28.7 us, with 1024 threads 31.5, 26 MB 32.4 and 32.8.
constexpr int kDecodeThreads = 1024;
constexpr int kDecodeThreadsSmall = 512;
// LDS for the payload slice, in words: what fits beside the tables
constexpr int kSmallWords = 61;
template <int THREADS> struct StageWords { static constexpr int kAll = THREADS >= 768 ? 768 * 46 : THREADS * kSmallWords; };
constexpr uint64_t kSmallSeats = kSmallWords * kDecodeThreadsSmall / 64;    // chunks of 8 bits per symbol that fit it: in practice, any
constexpr int kComputeUnits = 256;                 // MI355X
// encode: a group of the count and write passes has sixteen waves, four rounds of four chunks each.  With four waves of
// sixteen rounds a launch of fewer groups than the device holds at once waits for every round's loads in turn.  Count and
// write of 8 MB index streams (187 groups) 13.0 and 21.8 us, now 6.9 and 11.5; of 20 MB 12.7 and 27.5, now 8.5 and 19.7; of
// 51 MB 17.4 and 37.0, now 15.0 and 32.7 (eight waves: 9.6 and 22.3 at 20 MB, 16.8 and 32.8 at 51 MB).
constexpr int kGroup = 256;                        // chunks of a group
constexpr int kGroupThreads = 1024;
constexpr int kWaves = kGroupThreads / 64;
constexpr int kRounds = kGroup / kWaves / 4;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct Stream {                                    // what a launch is told of a stream
    uint8_t*  out;                                 // 256 lengths, chunks + 1 offsets, payload
    uint32_t* scratch;                             // the workspace: histogram, codes, group sums
    uint64_t* totals;                              // {stream bytes used, payload bits}
    const uint8_t* in;
    uint64_t  n;                                   // symbols (an upper bound when n_dev is set)
    const uint64_t* n_dev;                         // device: the symbol count, known only on the stream; or null
    StoredForm stored;                             // header: null outside the whole chain
    uint32_t  chunks, groups;
    uint32_t  hist_blocks;                         // workgroups of the histogram pass
};
struct Layout {                                    // where things are in the stream and in the workspace
    uint8_t*  len;                                 // [256]
    uint32_t* offsets;                             // [chunks + 1]
    uint32_t* payload;
    uint32_t* hist;                                // workspace: [256]
    uint32_t* table;                               // workspace: [256], the code from the top bit down | its length
    uint32_t* group_sums;                          // workspace: [groups]
    uint64_t* totals;
    const uint8_t* in;
    uint64_t  n;
    uint32_t  chunks, groups, hist_blocks;
    StoredForm stored;
};

__device__ __forceinline__ uint64_t chunks_for(uint64_t n) { return (n + 255u) >> 8; }

// The layout a kernel works with.  When the symbol count lives in device memory (it is the
// output of an earlier call on the same stream), the host has sized buffers and grids for an
// upper bound; the count itself, and what follows from it -- chunks, groups, where the payload
// starts -- is settled here, and workgroups beyond the real extent find nothing to do.
__device__ __forceinline__ Layout resolved(const Stream& given)
{
    Layout lay;
    lay.totals = given.totals;
    lay.in = given.in;
    lay.stored = given.stored;
    lay.n = given.n;
    lay.chunks = given.chunks;
    lay.groups = given.groups;
    lay.hist_blocks = given.hist_blocks;
    if (given.n_dev) {
        const uint64_t there = *given.n_dev;
        lay.n = there < given.n ? there : given.n;
        lay.chunks = (uint32_t)chunks_for(lay.n);
        lay.groups = (lay.chunks + 255u) >> 8;
        lay.hist_blocks = histogram_workgroups(lay.n);
    }
    lay.len = given.out;
    lay.offsets = reinterpret_cast<uint32_t*>(given.out + 256);
    lay.payload = lay.offsets + lay.chunks + 1;
    lay.hist = given.scratch;
    lay.table = lay.hist + 256;
    lay.group_sums = lay.table + 256;
    return lay;
}
// Where several histogram workgroups leave their 256 counts each, 16-byte aligned: in the payload's place, which is written after
// they have been read, and is longer than they are (a bit per symbol at least, where they are 1 KiB to 64 Ki symbols).
__device__ __forceinline__ uint32_t* hist_rows(const Layout& lay)
{
    return reinterpret_cast<uint32_t*>((reinterpret_cast<uintptr_t>(lay.payload) + 15u) & ~(uintptr_t)15u);
}

struct DecodeJob {
    const uint8_t*  len;
    const uint32_t* offsets;
    const uint32_t* payload;
    uint8_t*        out;
    uint64_t        n;                                        // symbols (an upper bound when n_dev is set)
    const uint64_t* n_dev;                                    // device: the symbol count; or null
    uint64_t        stream_bytes;                             // the valid prefix of the stream
    uint32_t        payload_words, chunks;
    uint32_t        blocks;                                   // workgroups of this stream
};

// Every pass serves up to kBatch streams (fh_batch.hpp); the per-stream passes take a workgroup per stream.

// ---- histogram ------------------------------------------------------------------------------------
// A workgroup clears and adds up 32 KiB of counters whatever it counts, so it has the most threads there are: at 51 MB in five
// streams 29 us with 256 threads (1340 workgroups), 18 us with 1024.  The code kernel adds up what the workgroups leave: with
// counters that they all add to, these had to be cleared by a launch before this one (encode and decode of 51 MB 125.4 us, 122.4 now).
template <typename Args>
__global__ __launch_bounds__(kHistThreads) void huffman_histogram_kernel(const Args batch)
{
    uint32_t block;
    const Layout lay = resolved(item_of(batch, blockIdx.x, block));
    if (block >= lay.hist_blocks) return;                     // workgroup-uniform: past the real extent
    const uint8_t* in = lay.in;
    const uint64_t n = lay.n;
    uint32_t* const counts = lay.hist_blocks == 1u ? lay.hist : hist_rows(lay) + 256u * block;
    // One copy of the histogram per LDS bank, the copies interleaved so that copy c of every bin lies in bank c:
    // lane l counts in copy l mod 32, and whatever the bytes are no two lanes of a half-wave meet in a bank
    // (bytes clustered around one value would otherwise serialise on the few bins they share).
    __shared__ uint32_t local[256][kHistCopies];
    for (int i = threadIdx.x; i < kHistCopies * 256; i += kHistThreads) (&local[0][0])[i] = 0u;
    __syncthreads();
    uint32_t* mine = &local[0][threadIdx.x & (kHistCopies - 1)];
    const uint64_t vectors = n >> 4;                          // `in` is 16-byte aligned
    const uint64_t stride = (uint64_t)lay.hist_blocks * kHistThreads;
    uint64_t v = (uint64_t)block * kHistThreads + threadIdx.x;
    u32x4 ahead = v < vectors ? reinterpret_cast<const u32x4*>(in)[v] : u32x4{0u, 0u, 0u, 0u};
    for (; v < vectors; v += stride) {
        const u32x4 w = ahead;
        if (v + stride < vectors) ahead = reinterpret_cast<const u32x4*>(in)[v + stride];   // in flight during the counting
        const uint32_t word[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int b = 0; b < 4; ++b) atomicAdd(&mine[((word[k] >> (8 * b)) & 0xffu) * kHistCopies], 1u);
    }
    if (block == 0) {                                         // the bytes after the last whole vector
        const uint64_t i = (vectors << 4) + threadIdx.x;
        if (threadIdx.x < 16 && i < n) atomicAdd(&mine[(uint32_t)in[i] * kHistCopies], 1u);
    }
    __syncthreads();
    // four neighbouring threads per bin, eight copies each; the fourth then has the bin's total
    static_assert(kHistThreads == 4 * 256 && kHistCopies == 32, "a thread adds up eight copies of a bin");
    const uint32_t bin = threadIdx.x >> 2, first = (threadIdx.x & 3u) * 8u;
    uint32_t total = 0;
#pragma unroll
    for (uint32_t c = 0; c < 8u; ++c) total += local[bin][first + ((c + bin) & 7u)];
    total = dpp_add<0x111, 0xf>(total);                       // row_shr:1, then 2: over the lane and the three below it
    total = dpp_add<0x112, 0xf>(total);
    if ((threadIdx.x & 3u) == 3u) counts[bin] = total;
}

// ---- code lengths and canonical codes ---------------------------------------------------------------
// The merges of the two-queue construction, one wave, as many of them at a time as do not depend on each other.
// Before a merge, let t be the sum of the two lightest nodes.  Every node made from now on weighs t at least and
// queues behind whatever weighs the same, so the nodes of weight <= t that are there now are taken in their present
// order, pair by pair, before any node made from now on: floor(k / 2) merges of one round, k being their number.
// Their order is the two queues merged by weight, a leaf first where weights are equal.  The wave looks at a window
// of 64 nodes of either queue, one per lane, so a round is limited to the first 64 nodes of that order (whatever
// comes behind a window cannot precede them).  A node's place in the order is its place in its own queue plus the
// nodes of the other queue that precede it.  Weights at least double from one round to the round after next, so the rounds are few (19 for the
// 256 symbols of an index stream, 12 for equal counts) where the merges one by one are up to 255 dependent steps
// of some 40 instructions each: the kernel took 57 us for the 249 merges of 250 symbols of like counts and takes 15.
constexpr uint32_t kNoNode = ~(uint32_t)0;
__device__ __forceinline__ uint32_t lane_value(uint32_t v, uint32_t from) { return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)from); }
__device__ __forceinline__ uint32_t smaller(uint32_t a, uint32_t b) { return a < b ? a : b; }
__device__ __forceinline__ uint32_t add_capped(uint32_t a, uint32_t b) { return __builtin_elementwise_add_sat(a, b); }
__device__ __forceinline__ uint32_t lane_below(uint32_t v)    // lanes 1..15 of a row: the lane before
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)kNoNode, (int)v, 0x111, 0xf, 0xf, false);
}

// weight[0 .. m): the leaves in rank order; weight[m .. 2m - 1) and parent[0 .. 2m - 2) are filled.  m >= 2.
__device__ __forceinline__ void merge_in_rounds(const uint32_t m, uint32_t* weight, uint16_t* parent, uint32_t* flag /* [64] */,
                                                const uint32_t lane)
{
    uint32_t next_leaf = 0, next_internal = m, made = m;      // wave-uniform
    while (made < 2u * m - 1u) {                              // a round makes a node at least
        const uint32_t leaf = next_leaf + lane, node = next_internal + lane;
        const bool is_leaf = leaf < m, is_node = node < made;
        const uint32_t of_leaf = is_leaf ? weight[leaf] : kNoNode, of_node = is_node ? weight[node] : kNoNode;
        // the smallest sum of two: leaf 0 + leaf 1 and node 0 + node 1 in lane 1, leaf 0 + node 0 in lane 0; sums with a
        // node that does not exist stay at kNoNode (two nodes exist, and all weights together are below 2^32)
        const uint32_t alike = smaller(add_capped(of_leaf, lane_below(of_leaf)), add_capped(of_node, lane_below(of_node)));
        const uint32_t t = smaller(lane_value(alike, 1), lane_value(add_capped(of_leaf, of_node), 0));
        const uint32_t leaves = (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(is_leaf && of_leaf <= t));
        const uint32_t nodes = (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(is_node && of_node <= t));
        const uint32_t all = leaves + nodes, taken = (all < 64u ? all : 64u) & ~1u;
        // Which places of the round's order the nodes of the queue with fewer candidates take: a candidate of the
        // other queue has its place by one compare and add per candidate of this one, its weight read from its lane.
        // (Four at a time: the weights behind the candidates are above t and precede no candidate.)
        const bool by_leaf = leaves < nodes;                  // wave-uniform
        const uint32_t theirs = by_leaf ? of_node : of_leaf, steps = by_leaf ? leaves : nodes, others = by_leaf ? nodes : leaves;
        uint32_t place = lane;
        if (by_leaf) {
            for (uint32_t k = 0; k < steps; k += 4)
#pragma unroll
                for (uint32_t j = 0; j < 4; ++j) place += lane_value(of_leaf, k + j) <= theirs ? 1u : 0u;   // a leaf first
        } else {
            for (uint32_t k = 0; k < steps; k += 4)
#pragma unroll
                for (uint32_t j = 0; j < 4; ++j) place += lane_value(of_node, k + j) < theirs ? 1u : 0u;
        }
        flag[lane] = 0u;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); // LDS operations of one wave complete in order
        if (lane < others && place < 64u) flag[place] = 1u;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        // lane l is place l of the order from here on
        const uint64_t marked = __builtin_amdgcn_ballot_w64(flag[lane] != 0u);
        const bool other = (marked >> lane) & 1u;
        const uint32_t marked_before = __builtin_amdgcn_mbcnt_hi((uint32_t)(marked >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)marked, 0u));
        const uint32_t index = other ? marked_before : lane - marked_before;      // in its queue's window
        const bool is_taken_node = other == by_leaf;
        const uint32_t at = (is_taken_node ? next_internal : next_leaf) + index;
        uint32_t w = 0;
        if (lane < taken) {
            w = weight[at];
            parent[at] = (uint16_t)(made + (lane >> 1));
        }
        const uint32_t sum = dpp_add<0x111, 0xf>(w);           // with the lane below
        if (lane < taken && (lane & 1u)) weight[made + (lane >> 1)] = sum;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const uint32_t gone = (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(lane < taken && !is_taken_node));
        next_leaf += gone;
        next_internal += taken - gone;
        made += taken >> 1;
    }
}

// the lanes whose code length, 24 at most, is this one's; every lane of the wave must be active
__device__ __forceinline__ uint64_t lanes_alike(uint32_t length)
{
    uint64_t same = ~(uint64_t)0;
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        const uint64_t has = __builtin_amdgcn_ballot_w64(((length >> k) & 1u) != 0u);
        same &= (length >> k) & 1u ? has : ~has;
    }
    return same;
}

// One workgroup per stream.  It runs once, alone on its compute unit, and every phase is a chain of dependent steps,
// so what counts is the length of the chains: the sixteen waves compare a quarter of the counts each for the ranks
// (four waves on a SIMD hide each other's latencies), threads 0..255 stand for the symbols elsewhere.  A 50 MB stream of 256
// clustered symbols: 19.1 us with the merges one by one, 16.2 now, of 250 symbols alike 57 and 15.3 (22 and 20 with the
// 64 counts of a quarter in registers at once: 88 bytes of scratch per lane).
constexpr int kCodeThreads = 1024;
template <typename Args>
__global__ __launch_bounds__(kCodeThreads) void huffman_code_kernel(const Args batch)
{
    const Layout lay = resolved(item_of(batch, blockIdx.x));
    // counts and weights are sums of at most 2^32 - 1 symbols: 32 bits hold them
    __shared__ __align__(16) uint32_t count[256];             // this round's counts, by symbol
    __shared__ uint32_t rank_of[256];
    __shared__ uint32_t weight[511];                          // leaves in rank order, then internal nodes as made
    __shared__ uint16_t parent[511];
    __shared__ uint32_t flag[64];                             // merges of a round: places that nodes of the one queue take
    __shared__ uint32_t up[2][511];
    __shared__ uint32_t in_wave[4][kMaxLen + 2];              // [w][k]: wave w's symbols that are unused (k = 0) / of length k
    __shared__ uint32_t first_code[64];
    __shared__ uint32_t bits_in_wave[4][2];
    __shared__ __align__(16) uint32_t of_rows[kCodeThreads / 64][256];     // the histogram workgroups' counts, as many sums as waves
    __shared__ uint32_t too_deep;
    const uint32_t thread = threadIdx.x, lane = thread & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(thread >> 6));
    const uint32_t s = thread & 255u, symbols = wave & 3u, quarter = wave >> 2;   // the wave's symbols: 64 symbols + lane
    const bool symbol = wave < 4u;
    uint32_t original = 0;
    if (lay.hist_blocks > 1u) {                               // workgroup-uniform; a wave a row at a time, four in flight
        const u32x4* rows = reinterpret_cast<const u32x4*>(hist_rows(lay)) + lane;
        u32x4 sum = {0u, 0u, 0u, 0u};
        constexpr uint32_t kAtOnce = 4, kStep = kCodeThreads / 64;
        for (uint32_t r = wave; r < lay.hist_blocks; r += kAtOnce * kStep) {
            u32x4 got[kAtOnce];
#pragma unroll
            for (uint32_t k = 0; k < kAtOnce; ++k) got[k] = r + k * kStep < lay.hist_blocks ? rows[64u * (r + k * kStep)] : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
            for (uint32_t k = 0; k < kAtOnce; ++k) sum += got[k];
        }
        reinterpret_cast<u32x4*>(of_rows[wave])[lane] = sum;
        __syncthreads();
#pragma unroll
        for (uint32_t w = 0; w < kStep; ++w) original += of_rows[w][s];
    } else if (lay.hist_blocks == 1u) {
        original = lay.hist[s];
    }
    uint32_t c = original, my_length = 0;
    for (;;) {                                                // workgroup-uniform; counts halve, so it ends
        if (symbol) {
            count[s] = c;
            rank_of[s] = 0u;
            const uint64_t unused = __builtin_amdgcn_ballot_w64(c == 0u);
            if (lane == 0) in_wave[wave][0] = (uint32_t)__popcll(unused);
            if (s == 0) too_deep = 0u;
        }
        __syncthreads();
        const uint32_t m = 256u - (in_wave[0][0] + in_wave[1][0] + in_wave[2][0] + in_wave[3][0]);   // used symbols
        // symbols before this one by (count, symbol), of this thread's quarter.  On equal counts those of a quarter
        // below precede, those of one above do not: "<=" is "< c + 1", which needs a count below 2^32 - 1, and one
        // symbol alone can have that many: any count above 0 ranks it last.
        {
            const uint32_t key = c < ~0u ? c : c - 1u;
            const uint32_t bound = quarter < symbols ? key + 1u : key;
            uint32_t before = 0;                              // sixteen counts at a time: all 64 at once spill
            const u32x4* const theirs = reinterpret_cast<const u32x4*>(&count[64u * quarter]);
            if (quarter == symbols) {
#pragma unroll 1
                for (int g = 0; g < 4; ++g) {
                    const u32x4 four[4] = {theirs[4 * g], theirs[4 * g + 1], theirs[4 * g + 2], theirs[4 * g + 3]};
#pragma unroll
                    for (int k = 0; k < 16; ++k) before += four[k >> 2][k & 3] < key + ((uint32_t)(16 * g + k) < lane ? 1u : 0u) ? 1u : 0u;
                }
            } else {
#pragma unroll 1
                for (int g = 0; g < 4; ++g) {
                    const u32x4 four[4] = {theirs[4 * g], theirs[4 * g + 1], theirs[4 * g + 2], theirs[4 * g + 3]};
#pragma unroll
                    for (int k = 0; k < 16; ++k) before += four[k >> 2][k & 3] < bound ? 1u : 0u;
                }
            }
            atomicAdd(&rank_of[s], before);
        }
        __syncthreads();
        const uint32_t rank = rank_of[s] - (256u - m);        // the unused ones come first: taken off again
        if (symbol && c != 0) weight[rank] = c;
        __syncthreads();
        const uint32_t mm = (uint32_t)__builtin_amdgcn_readfirstlane((int)m);
        if (wave == 0 && mm > 1u) merge_in_rounds(mm, weight, parent, flag, lane);
        __syncthreads();
        // Depths by pointer doubling: up[node] = steps << 16 | the node that many steps above it, doubled five times,
        // so that a leaf that has not arrived at the root is more than 32 deep and the code is over the limit anyway.
        const uint32_t root = m ? 2u * m - 2u : 0u;
        if (thread < 511u) up[0][thread] = thread < root ? 0x10000u | parent[thread] : thread;
        __syncthreads();
#pragma unroll
        for (int step = 0; step < 5; ++step) {
            if (thread < 511u) {
                const uint32_t here = up[step & 1][thread];
                up[~step & 1][thread] = (here & 0xffff0000u) + up[step & 1][here & 0xffffu];
            }
            __syncthreads();
        }
        if (symbol && c != 0) {
            const uint32_t mine = up[1][rank];
            my_length = m == 1u ? 1u : (mine & 0xffffu) == root ? mine >> 16 : 255u;
            if (my_length > (uint32_t)kMaxLen) too_deep = 1u;
        }
        __syncthreads();
        if (!too_deep) break;
        if (c != 0) c = (c + 1) >> 1;
        __syncthreads();                                      // everyone has read `too_deep` before it is written again
    }
    // canonical codes: by increasing (length, symbol); a symbol's place among those of its length from lane masks
    // inside the wave plus the counts of the waves below.  Payload bits: every symbol's count times its length (the
    // counts as they were), the counts' halves apart so that a wave's sums fit 32 bits.
    uint32_t before = 0;
    if (symbol) {
        if (lane <= (uint32_t)kMaxLen + 1u) in_wave[wave][lane] = 0u;
        const uint64_t same = lanes_alike(my_length);
        before = __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); // LDS operations of one wave complete in order
        if (my_length && before == 0u) in_wave[wave][my_length] = (uint32_t)__popcll(same);
        const uint32_t low = wave_inclusive_scan((original & 0xffffu) * my_length), high = wave_inclusive_scan((original >> 16) * my_length);
        if (lane == 63u) { bits_in_wave[wave][0] = low; bits_in_wave[wave][1] = high; }
    }
    __syncthreads();
    if (wave == 0) {
        // first code of length k = sum over the shorter lengths j of their symbols << (k - j); scaled by 2^(24 - k) that
        // is a prefix sum (at most 2^24, Kraft's sum being at most 1)
        const bool a_length = lane >= 1u && lane <= (uint32_t)kMaxLen;
        const uint32_t of_length = a_length ? in_wave[0][lane] + in_wave[1][lane] + in_wave[2][lane] + in_wave[3][lane] : 0u;
        const uint32_t scaled = a_length ? of_length << ((uint32_t)kMaxLen - lane) : 0u;
        const uint32_t shorter = wave_inclusive_scan(scaled) - scaled;
        first_code[lane] = a_length ? shorter >> ((uint32_t)kMaxLen - lane) : 0u;
        if (lane == 0) {
            uint64_t bits = 0;
            for (int w = 0; w < 4; ++w) bits += bits_in_wave[w][0] + ((uint64_t)bits_in_wave[w][1] << 16);
            lay.totals[1] = bits;
        }
    }
    __syncthreads();
    if (symbol) {
        if (my_length) for (uint32_t w = 0; w < wave; ++w) before += in_wave[w][my_length];
        const uint32_t code = my_length ? first_code[my_length] + before : 0u;
        lay.len[s] = (uint8_t)my_length;
        lay.table[s] = my_length ? (code << (32u - my_length)) | my_length : 0u;
    }
}

// the symbols of a chunk, 16 at a time; `valid` of them exist
__device__ __forceinline__ void load_symbols(const uint8_t* in, uint64_t first, uint32_t valid, uint32_t (&word)[4])
{
    if (valid >= 16u) {
        const u32x4 w = *reinterpret_cast<const u32x4*>(in + first);
        word[0] = w.x; word[1] = w.y; word[2] = w.z; word[3] = w.w;
        return;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        word[k] = 0u;
#pragma unroll
        for (int b = 0; b < 4; ++b)
            if ((uint32_t)(4 * k + b) < valid) word[k] |= (uint32_t)in[first + 4 * k + b] << (8 * b);
    }
}

__device__ __forceinline__ uint32_t larger(uint32_t a, uint32_t b) { return a > b ? a : b; }
// the largest of the values of the lanes up to this one; every lane of the wave must be active
template <int CTRL, int ROW_MASK> __device__ __forceinline__ uint32_t dpp_larger(uint32_t v)
{
    return larger(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xf, false));
}
__device__ __forceinline__ uint32_t wave_inclusive_max(uint32_t v)
{
    v = dpp_larger<0x111, 0xf>(v);                            // as the sums of fh_scan.hpp
    v = dpp_larger<0x112, 0xf>(v);
    v = dpp_larger<0x114, 0xf>(v);
    v = dpp_larger<0x118, 0xf>(v);
    v = dpp_larger<0x142, 0xa>(v);
    v = dpp_larger<0x143, 0xc>(v);
    return v;
}

// exclusive prefix over the workgroup of one value per thread; all = the workgroup's total
__device__ __forceinline__ uint32_t workgroup_exclusive_scan(uint32_t mine, uint32_t* lds /* [4] */, uint32_t* all)
{
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint32_t inc = wave_inclusive_scan(mine);
    if (lane == 63u) lds[wave] = inc;
    __syncthreads();
    uint32_t before = 0, total = 0;
#pragma unroll
    for (int v = 0; v < kThreads / 64; ++v) {
        const uint32_t t = lds[v];
        if ((uint32_t)v < wave) before += t;
        total += t;
    }
    __syncthreads();
    *all = total;
    return before + inc - mine;
}

// ---- count: words per chunk, sums per group -------------------------------------------------------
// Sixteen lanes share a chunk: a wave reads four consecutive chunks, 1 KiB, with one 16-byte load per lane --
// whole cache lines, each fetched once -- and does so for its 16 chunks in four rounds, all in flight at once.  (A thread per chunk,
// walking its 256 bytes alone, asks for 16 bytes of every line its wave touches in a round and finds the rest
// gone from the cache when it comes back: measured, that read 1.2 times the input here and 2.9 times in the
// write pass.)
struct PieceOfChunk {                              // what a lane reads in one round
    uint32_t chunk;                                // the chunk (of the stream), which may not exist
    uint32_t have;                                 // symbols of its 16 that exist: 0 .. 16
    uint64_t first;                                // index of the first of them
};
__device__ __forceinline__ PieceOfChunk piece_of(const Layout& lay, uint32_t chunk0, uint32_t lane)     // the round's first chunk
{
    PieceOfChunk p;
    p.chunk = chunk0 + (lane >> 4);
    p.first = (uint64_t)p.chunk * kChunk + (lane & 15u) * 16u;
    p.have = p.first >= lay.n ? 0u : lay.n - p.first < 16u ? (uint32_t)(lay.n - p.first) : 16u;
    return p;
}
// does every lane of the wave have all its 16 symbols in this round?  (wave-uniform, from scalar values)
__device__ __forceinline__ bool round_is_whole(const Layout& lay, uint32_t chunk0)
{
    return ((uint64_t)chunk0 + 4u) * kChunk <= lay.n;
}
// sum over the 16 lanes that share a chunk, in the last of them (row shifts: a row of the wave is those 16 lanes)
__device__ __forceinline__ uint32_t sum_to_lane_15_of_row(uint32_t v)
{
    v = dpp_add<0x111, 0xf>(v);
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    v = dpp_add<0x118, 0xf>(v);
    return v;                                                 // inclusive prefix inside the row
}

template <typename Args>
__global__ __launch_bounds__(kGroupThreads) void huffman_count_kernel(const Args batch)
{
    uint32_t group;
    const Layout lay = resolved(item_of(batch, blockIdx.x, group));
    if (group >= lay.groups) return;                          // workgroup-uniform: past the real extent
    __shared__ uint8_t len[256];
    __shared__ uint32_t lds[kWaves];
    if (threadIdx.x < 256u) len[threadIdx.x] = (uint8_t)(lay.table[threadIdx.x] & 0xffu);
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t wave_chunk = group * kGroup + wave * (4u * kRounds);
    uint32_t closed = 0;                                      // words of the chunks this lane closed (lanes 15, 31, 47, 63)
    uint32_t word[kRounds][4];
#pragma unroll
    for (int k = 0; k < kRounds; ++k) {
        const uint32_t chunk0 = wave_chunk + 4u * k;
        const PieceOfChunk p = piece_of(lay, chunk0, lane);
        if (round_is_whole(lay, chunk0)) {
            const u32x4 w = *reinterpret_cast<const u32x4*>(lay.in + p.first);
            word[k][0] = w.x; word[k][1] = w.y; word[k][2] = w.z; word[k][3] = w.w;
        } else {
            word[k][0] = word[k][1] = word[k][2] = word[k][3] = 0u;
            if (p.have) load_symbols(lay.in, p.first, p.have, word[k]);
        }
    }
    __syncthreads();                                          // `len`, once the symbols have been asked for
#pragma unroll
    for (int k = 0; k < kRounds; ++k) {
        const uint32_t chunk0 = wave_chunk + 4u * k;
        const PieceOfChunk p = piece_of(lay, chunk0, lane);
        uint32_t bits = 0;
        if (round_is_whole(lay, chunk0)) {
#pragma unroll
            for (int j = 0; j < 16; ++j) bits += len[(word[k][j >> 2] >> (8 * (j & 3))) & 0xffu];
        } else {
#pragma unroll
            for (int j = 0; j < 16; ++j)
                if ((uint32_t)j < p.have) bits += len[(word[k][j >> 2] >> (8 * (j & 3))) & 0xffu];
        }
        const uint32_t of_chunk = sum_to_lane_15_of_row(bits);
        if ((lane & 15u) == 15u && p.chunk < lay.chunks) {
            const uint32_t words = (of_chunk + 31u) >> 5;
            lay.offsets[p.chunk] = words;                     // becomes the chunk's offset in the write pass
            closed += words;
        }
    }
    const uint32_t of_wave = wave_inclusive_scan(closed);
    if (lane == 63u) lds[wave] = of_wave;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t sum = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) sum += lds[w];
        lay.group_sums[group] = sum;
    }
}

// ---- scan of the group sums (in place, exclusive); the stream's size --------------------------------------
// `words`: of the stream's payload; one thread
__device__ __forceinline__ void leave_size(const Layout& lay, uint32_t words)
{
    const uint64_t bytes = 256u + 4ull * (lay.chunks + 1ull) + 4ull * words;
    lay.offsets[lay.chunks] = words;
    lay.totals[0] = bytes;
    const StoredForm& f = lay.stored;
    if (f.header) f.header[6] = f.fixed_bytes + f.header[0] * f.value_size + bytes;
}
__global__ __launch_bounds__(kThreads) void huffman_scan_kernel(const Batch<Stream> batch)
{
    const Layout lay = resolved(batch.item[blockIdx.x]);
    __shared__ uint32_t lds[4];
    uint32_t carry = 0;
    for (uint32_t base = 0; base < lay.groups; base += kThreads) {         // workgroup-uniform trip count
        const uint32_t i = base + threadIdx.x;
        const uint32_t mine = i < lay.groups ? lay.group_sums[i] : 0u;
        uint32_t total;
        const uint32_t before = workgroup_exclusive_scan(mine, lds, &total);
        if (i < lay.groups) lay.group_sums[i] = carry + before;
        carry += total;
    }
    if (threadIdx.x == 0) leave_size(lay, carry);
}

// ---- write: offsets and payload -------------------------------------------------------------------
// The same sharing as in the count pass: a wave codes four consecutive chunks per round, sixteen lanes to a chunk,
// each lane its 16 symbols.  A lane looks its 16 codes up, the lengths are prefix-summed over the chunk's lanes,
// and the lane then puts its bits where they belong in the wave's staging area in LDS -- whole words as they fill
// up, with an OR, since the first and the last word of a lane's run are shared with its neighbours.  The four
// chunks are one contiguous piece of the payload (each starts on a word); the wave copies it out with consecutive
// lanes on consecutive words and leaves the area cleared for the next round.  A chunk is at most 192 words
// (24 bits per symbol), so the area fits whatever the stream holds.
// What bounds the pass is the vector instructions of a lane's chain: with two symbols a step, a half of the steps, 51 MB
// of index streams take 27.9 us, 32.4 with one; 20 and 8 MB 17.0 and 10.0, with one 20.0 and 11.4.
constexpr int kRoundWordsMax = 4 * kChunkWordsMax;          // 768 words per wave
constexpr uint32_t kCodeMask = ~(uint32_t)0xffu;            // of an entry of the table: codes have 24 bits at most

template <bool SCANNED, typename Args>
__global__ __launch_bounds__(kGroupThreads) void huffman_write_kernel(const Args batch)
{
    uint32_t group;
    const Layout lay = resolved(item_of(batch, blockIdx.x, group));
    if (group >= lay.groups) {                                // workgroup-uniform: past the real extent
        if (!SCANNED && lay.groups == 0u && group == 0u && threadIdx.x == 0) leave_size(lay, 0u);
        return;
    }
    __shared__ uint32_t table[256];
    __shared__ uint32_t lds[4], below[kWaves];
    __shared__ uint32_t chunk_at[kGroup + 4];                 // word offset of every chunk inside the group's slice; [256..]: the total
    __shared__ uint32_t area[kWaves][kRoundWordsMax + 4];
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // the first four waves have a thread per chunk of the group, and per symbol
    const uint32_t chunk = group * kGroup + threadIdx.x;
    const bool live = threadIdx.x < (uint32_t)kGroup && chunk < lay.chunks;
    const uint32_t words = live ? lay.offsets[chunk] : 0u;
    uint32_t before_group = 0;
    if constexpr (!SCANNED) {
        for (uint32_t g = threadIdx.x; g < group; g += kGroupThreads) before_group += lay.group_sums[g];
    }
    if (threadIdx.x < 256u) table[threadIdx.x] = lay.table[threadIdx.x];
    const uint32_t upto = wave_inclusive_scan(words);
    if (wave < 4u && lane == 63u) lds[wave] = upto;
    if constexpr (!SCANNED) {
        const uint32_t of_wave = wave_inclusive_scan(before_group);
        if (lane == 63u) below[wave] = of_wave;
    }
    uint32_t* mine = area[wave];
    for (uint32_t w = lane; w < (uint32_t)kRoundWordsMax + 4u; w += 64u) mine[w] = 0u;
    __syncthreads();
    uint32_t base = 0;                                        // words of the groups before this one
    if constexpr (SCANNED) base = lay.group_sums[group];
    else {
#pragma unroll
        for (int w = 0; w < kWaves; ++w) base += below[w];
    }
    if (wave < 4u) {
        uint32_t before = upto - words;
        for (uint32_t w = 0; w < wave; ++w) before += lds[w];
        if (live) lay.offsets[chunk] = base + before;
        chunk_at[threadIdx.x] = before;
        if (threadIdx.x < 4u) chunk_at[kGroup + threadIdx.x] = lds[0] + lds[1] + lds[2] + lds[3];
    }
    if (!SCANNED && group + 1u == lay.groups && threadIdx.x == 0) leave_size(lay, base + lds[0] + lds[1] + lds[2] + lds[3]);
    __syncthreads();
    uint32_t* slice = lay.payload + base;
    const auto ask = [&](uint32_t round, uint32_t (&to)[4]) {
        const uint32_t first = group * kGroup + wave * (4u * kRounds) + round * 4u;
        const PieceOfChunk p = piece_of(lay, first, lane);
        if (round_is_whole(lay, first)) {
            const u32x4 w = *reinterpret_cast<const u32x4*>(lay.in + p.first);
            to[0] = w.x; to[1] = w.y; to[2] = w.z; to[3] = w.w;
        } else {
            to[0] = to[1] = to[2] = to[3] = 0u;
            if (p.have) load_symbols(lay.in, p.first, p.have, to);
        }
    };
    uint32_t ahead[4];
    ask(0, ahead);
    for (uint32_t round = 0; round < (uint32_t)kRounds; ++round) {
        const uint32_t chunk0 = wave * (4u * kRounds) + round * 4u;              // of the group: the first of this round's four
        const PieceOfChunk p = piece_of(lay, group * kGroup + chunk0, lane);
        const bool whole = round_is_whole(lay, group * kGroup + chunk0);
        const uint32_t run_at = chunk_at[chunk0], run = chunk_at[chunk0 + 4u] - run_at;   // wave-uniform
        if (run == 0u) break;                                 // nothing from here on (the stream has ended)
        // the lane's codes; those of the next round are asked for before these are coded
        const uint32_t word[4] = {ahead[0], ahead[1], ahead[2], ahead[3]};
        if (round + 1u < (uint32_t)kRounds) ask(round + 1u, ahead);
        uint32_t e[16];                                       // a symbol that does not exist: 0
        if (whole) {
#pragma unroll
            for (int j = 0; j < 16; ++j) e[j] = table[(word[j >> 2] >> (8 * (j & 3))) & 0xffu];
        } else {
#pragma unroll
            for (int j = 0; j < 16; ++j) e[j] = (uint32_t)j < p.have ? table[(word[j >> 2] >> (8 * (j & 3))) & 0xffu] : 0u;
        }
        // two symbols as one code of up to 32 bits, from the top bit down: half the steps of the chain below
        uint32_t code[8], length[8], bits = 0, longest = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            length[j] = (e[2 * j] + e[2 * j + 1]) & 0xffu;
            code[j] = (e[2 * j] & kCodeMask) | ((e[2 * j + 1] & kCodeMask) >> (e[2 * j] & 31u));
            bits += length[j];
            longest = longest > length[j] ? longest : length[j];
        }
        // where the lane's bits start: its chunk's word offset inside the round, then the lanes before it in the chunk
        const uint32_t start = ((chunk_at[chunk0 + (lane >> 4)] - run_at) << 5) + (sum_to_lane_15_of_row(bits) - bits);
        uint32_t* at = mine + (start >> 5);                   // the word being filled
        uint32_t filled = start & 31u;                        // bits of it that are taken
        uint32_t now = 0;                                     // it, as far as it is this lane's
        const auto put = [&](uint32_t c, uint32_t l) {        // l <= 32
            now |= c >> filled;
            const uint32_t rest = __builtin_amdgcn_alignbit(c, 0u, filled);      // c << (32 - filled); 0 when filled is 0
            filled += l;
            if (filled >= 32u) {
                atomicOr(at, now);
                ++at;
                now = rest;
                filled -= 32u;
            }
        };
        if (__builtin_amdgcn_ballot_w64(longest > 32u) == 0u) {
#pragma unroll
            for (int j = 0; j < 8; ++j) put(code[j], length[j]);
        } else {                                              // some lane's two codes together do not fit a word
#pragma unroll
            for (int j = 0; j < 16; ++j) put(e[j] & kCodeMask, e[j] & 0xffu);
        }
        if (filled) atomicOr(at, now);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");     // LDS operations of one wave complete in order
        for (uint32_t w = lane; w < run; w += 64u) {
            slice[run_at + w] = mine[w];
            mine[w] = 0u;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
}

// What a stream's codes are decoded with when the lookup table does not have them, in LDS.
struct LongCodes {
    uint32_t last[32];                                        // [k]: the largest window that starts with a code of length <= k
    uint32_t place[32];                                       // [k]: place in `sorted` of the first code of length k, less that code
    uint8_t  sorted[256];                                     // symbols by (length, symbol)
};

// An entry of the decoder's tables: symbol << 8 | 32 - length; 0 where there is none.  With what the code leaves of a
// word at the bottom, the entry as it is read is the shift amount that moves the stream up (drop_code).
__device__ __forceinline__ uint32_t entry_of(uint32_t symbol, uint32_t length) { return (symbol << 8) | (32u - length); }
__device__ __forceinline__ uint32_t symbols_in(const uint32_t (&e)[4])                              // a byte each
{
    return __builtin_amdgcn_perm(__builtin_amdgcn_perm(e[3], e[2], 0x05010501u), __builtin_amdgcn_perm(e[1], e[0], 0x05010501u), 0x05040100u);
}
__device__ __forceinline__ uint32_t length_in(uint32_t entry) { return 32u - (entry & 0xffu); }     // 32 where there is none

// The next 64 bits of the stream, the next one on top.  Two words and 32-bit shifts: a 64-bit shift whose amount the
// compiler put into the last register of a wave's 128 was seen to shift by register 0 instead, on some waves.
struct Ahead {
    uint32_t high, low;
};
// low word of high:low >> by; by mod 32 counts
__device__ __forceinline__ uint32_t align_right(uint32_t high, uint32_t low, uint32_t by) { return __builtin_amdgcn_alignbit(high, low, by); }
__device__ __forceinline__ Ahead drop_code(const Ahead& a, uint32_t entry)                         // an entry that exists
{
    return Ahead{align_right(a.high, a.low, entry), a.low << ((0u - entry) & 31u)};
}

// The entry of a code longer than SHORT bits that is on top of the stream.
// Canonical codes grow with their length, so the 32-bit windows that start with a code of length <= k are those up
// to last[k]: the length of the code on top is one more than the number of those bounds that the window exceeds -- a
// compare and an add per length, the bounds (the same for the whole workgroup) in scalar registers -- and its place
// among the symbols sorted by (length, symbol) is its value plus `place` of its length.  `top`: the next
// 32 bits of the stream.
template <int SHORT> struct LongRegs {
    uint32_t last[kMaxLen - SHORT - 1];            // [i]: the largest window that starts with a code of length <= SHORT + 1 + i
};
template <int SHORT>
__device__ __forceinline__ LongRegs<SHORT> long_regs(const LongCodes* t)
{
    LongRegs<SHORT> r;
#pragma unroll
    for (int i = 0; i < kMaxLen - SHORT - 1; ++i) r.last[i] = (uint32_t)__builtin_amdgcn_readfirstlane((int)t->last[SHORT + 1 + i]);
    return r;
}
// its entry; the length is SHORT + 1 at least, whatever the tables say
template <int SHORT>
__device__ __forceinline__ uint32_t decode_long(uint32_t top, const LongRegs<SHORT>& r, const LongCodes* t)
{
    uint32_t length = SHORT + 1;
#pragma unroll
    for (int i = 0; i < kMaxLen - SHORT - 1; ++i) length += top > r.last[i] ? 1u : 0u;
    return entry_of(t->sorted[((top >> (32u - length)) + t->place[length]) & 0xffu], length);
}

// The lookup table of a stream, indexed by the stream's next bits.  Canonical codes grow with their length, so the codes
// longer than kFastBits are the upper end of the code space: the windows whose first kFastBits bits are `from` or more.
// Up to there an entry stands for kFastBits bits, behind it for kFastBits + extra, and the index is the larger of the two
// readings: top >> (32 - kFastBits), and (top >> shift) + add with shift = 32 - kFastBits - extra, add = from - (from << extra).
// (Below `from` the second falls behind the first by a step of the finer reading where the first falls by one of the coarser.)
// `extra` is as large as the table's room allows, the longest code and kReach at most; 0 makes both readings the same.
// Entries of codes longer still are 0: these walk the lengths.  One read and no branch for a code of either kind: as two
// tables, the second read where the first had nothing, some lane of a wave took the branch at two symbols in five
// (12 bits, 51 MB of index streams), 400 cycles for all of them; those streams decode in 45.5 us, 50.6 with two tables.
constexpr int kFastBits = 12;
constexpr int kSecondEntries = 2048;               // room behind 1 << kFastBits entries
constexpr int kTableEntries = (1 << kFastBits) + kSecondEntries;
constexpr uint32_t kReach = 21;                    // bits that a lookup looks at, at most: three codes fit a window of 64
struct Lookup {
    const uint16_t*  table;
    const LongCodes* tables;
    uint32_t         shift;
    int32_t          add;
};
__device__ __forceinline__ uint32_t table_index(uint32_t shift, int32_t add, uint32_t top)
{
    const int32_t coarse = (int32_t)(top >> (32 - kFastBits)), fine = (int32_t)(top >> shift) + add;
    return (uint32_t)(coarse > fine ? coarse : fine);
}

// What a thread has decoded goes out kBurst vectors at a time.  LINES: half of a cache line waits for the other half, and the
// line's stores go out back to back, so that it is complete in the L2 before it can be evicted.
template <bool LINES> struct Output {
    uint8_t* dst;
    u32x4    first_half[kBurst];
    __device__ __forceinline__ void store(uint32_t at, uint32_t valid, const u32x4 (&piece)[kBurst])
    {
        if constexpr (LINES) {
            const bool second = (at / (16 * kBurst)) % 2u != 0u;
            if (!second && at + 16 * kBurst < valid) {
#pragma unroll
                for (int v = 0; v < kBurst; ++v) first_half[v] = piece[v];
                return;
            }
            if (second) {
#pragma unroll
                for (int v = 0; v < kBurst; ++v) *reinterpret_cast<u32x4*>(dst + at - 16 * (kBurst - v)) = first_half[v];
            }
        }
#pragma unroll
        for (int v = 0; v < kBurst; ++v) {
            const uint32_t i = at + 16u * v;
            if (i + 16 <= valid) {
                *reinterpret_cast<u32x4*>(dst + i) = piece[v];
            } else if (i < valid) {
                const uint32_t w[4] = {piece[v].x, piece[v].y, piece[v].z, piece[v].w};
                for (uint32_t b = 0; i + b < valid; ++b) dst[i + b] = (uint8_t)(w[b >> 2] >> (8 * (b & 3u)));
            }
        }
    }
};
// One chunk: `valid` symbols from the words first_word, next_word(1), next_word(2), ... to dst (16-byte aligned).
// A lane in three or four takes a word at any step, so the wave steps aside for it nearly always: the word that it takes then
// has been read before, and only the table is waited for (51 MB, half of it noise, 107 us with the word read when it is
// needed, 89 now; with eight vectors held back, the word read ahead alone 102).
template <typename NextWord>
__device__ __forceinline__ void decode_chunk(uint32_t valid, uint8_t* dst, const Lookup look, uint32_t first_word, NextWord next_word)
{
    const LongRegs<kFastBits> longer = long_regs<kFastBits>(look.tables);
    uint32_t word = first_word, taken = 1;                    // the word that comes behind `next`; words taken up to it
    Ahead next = {0u, 0u};
    uint32_t have = 0;                                        // bits of it that are there
    Output<true> out;
    out.dst = dst;
#pragma unroll 1
    for (uint32_t half = 0; half < valid; half += 16 * kBurst) {
        u32x4 piece[kBurst];
#pragma unroll
        for (int v = 0; v < kBurst; ++v) {
            uint32_t sixteen[4];
            if (half + 16u * v >= valid) { piece[v] = u32x4{0u, 0u, 0u, 0u}; continue; }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint32_t e[4];
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    if (have < 32u) {                         // (the low word is used up: 32 bits are enough for any code)
                        next.high |= word >> have;
                        next.low = align_right(word, 0u, have);
                        have += 32u;
                        word = next_word(taken);
                        ++taken;
                    }
                    e[b] = look.table[table_index(look.shift, look.add, next.high)];
                    if (__builtin_expect(e[b] == 0u, 0)) e[b] = decode_long<kFastBits>(next.high, longer, look.tables);
                    next = Ahead{align_right(next.high, next.low, e[b]), align_right(next.low, 0u, e[b])};
                    have -= length_in(e[b]);
                }
                sixteen[q] = symbols_in(e);
            }
            piece[v] = u32x4{sixteen[0], sixteen[1], sixteen[2], sixteen[3]};
        }
        out.store(half, valid, piece);
    }
}

// The same from words in LDS.  What a symbol costs is the chain from one table read to the next, so four symbols come
// from one 64-bit window of the stream, kept in registers: a table read, a shift by what it says.  Three codes that the table has
// fit it; the fourth may find too few bits left (rare), and codes that walk the lengths (rarer) start a new window behind
// them.  The words of the next window are requested before the fourth symbol's table read: its code moves the
// window's first word by one at most, so four words hold it either way.
// A window at bit `pos` starts in word (pos - 1) / 32, rounded down, so that its shift is 0 .. 31: at the chunk's first
// bit that is words[-1], shifted out whole.
struct Window {
    uint32_t w0, w1, w2;
};
__device__ __forceinline__ int32_t window_word(uint32_t pos) { return (int32_t)(pos - 1u) >> 5; }
__device__ __forceinline__ Ahead window_bits(const Window& w, uint32_t pos)
{
    return Ahead{align_right(w.w0, w.w1, 0u - pos), align_right(w.w1, w.w2, 0u - pos)};
}
// FINE: the table has finer entries.  Without (streams of few symbols: no code is longer than kFastBits, or too many are) an index is one
// shift: 134 MB of three symbols 76.1 -> 69.2 us, of one 92.0 -> 84.7 (74.1 and 87.8 with two tables).
template <bool LINES, bool FINE>
__device__ __forceinline__ void decode_chunk_staged(uint32_t valid, uint8_t* dst, const Lookup look, const uint32_t* words)
{
    const LongRegs<kFastBits> longer = long_regs<kFastBits>(look.tables);
    const uint32_t room = 64u - (32u - look.shift);           // bits of a window that may be gone before a lookup
    uint32_t pos = 0;                                         // bits of the chunk consumed
    Window w = {0u, words[0], words[1]};
    Output<LINES> out;
    out.dst = dst;
#pragma unroll 1
    for (uint32_t half = 0; half < valid; half += 16 * kBurst) {
        u32x4 piece[kBurst];
#pragma unroll
        for (int v = 0; v < kBurst; ++v) {
            uint32_t sixteen[4];
            if (half + 16u * v >= valid) { piece[v] = u32x4{0u, 0u, 0u, 0u}; continue; }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                Ahead next = window_bits(w, pos);
                uint32_t window = pos;                        // where it starts
                const auto new_window = [&](uint32_t from) {
                    const uint32_t* first = words + window_word(from);
                    window = from;
                    next = window_bits(Window{first[0], first[1], first[2]}, from);
                };
                uint32_t e[4];
                uint32_t sum = 0;                             // of the entries, whose low bytes are 32 - length: below 128 together
                int32_t at = 0;                               // where the fourth symbol's window starts
                uint32_t ahead[4];
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    if (b == 3) {
                        const uint32_t here = pos + 96u - (sum & 0xffu);
                        at = window_word(here);
#pragma unroll
                        for (int k = 0; k < 4; ++k) ahead[k] = words[at + k];
                        if (FINE && __builtin_expect(here - window > room, 0)) next = window_bits(Window{ahead[0], ahead[1], ahead[2]}, here);
                    }
                    const Ahead before = next;
                    e[b] = look.table[FINE ? table_index(look.shift, look.add, before.high) : before.high >> (32 - kFastBits)];
                    next = drop_code(before, e[b]);           // (put right below where there is no entry)
                    if (__builtin_expect(e[b] == 0u, 0)) {
                        const uint32_t here = pos + 32u * b - (sum & 0xffu);
                        next = before;
                        if (b > 0 && window + 64u - here < (uint32_t)kMaxLen) new_window(here);
                        e[b] = decode_long<kFastBits>(next.high, longer, look.tables);
                        if (b < 3) new_window(here + length_in(e[b]));
                    }
                    sum += e[b];
                }
                pos += 128u - (sum & 0xffu);
                const bool crossed = window_word(pos) != at;  // a code has at most 24 bits
                w = Window{crossed ? ahead[1] : ahead[0], crossed ? ahead[2] : ahead[1], crossed ? ahead[3] : ahead[2]};
                sixteen[q] = symbols_in(e);
            }
            piece[v] = u32x4{sixteen[0], sixteen[1], sixteen[2], sixteen[3]};
        }
        out.store(half, valid, piece);
    }
}

// ---- decode -------------------------------------------------------------------------------------------
// The stream may be foreign: the tables are built from whatever the 256 length bytes say
// (lengths above 24 count as unused), reads of payload words are bounded by the stream's size
// (words outside read as zero), and every loop is bounded by the symbol count.
template <int kDecodeThreads, bool LINES, typename Args>
__global__ __launch_bounds__(kDecodeThreads) void huffman_decode_kernel(const Args batch)
{
    constexpr int kStageWords = StageWords<kDecodeThreads>::kAll;
    uint32_t block;
    const DecodeJob& job = item_of(batch, blockIdx.x, block);
    const uint8_t* len_in = job.len;
    const uint32_t* offsets = job.offsets;
    const uint32_t* payload = job.payload;
    uint32_t payload_words = job.payload_words, chunks = job.chunks;
    uint64_t n = job.n;
    if (job.n_dev) {                                          // the count is on the stream: settle what follows from it
        const uint64_t there = *job.n_dev;
        n = there < job.n ? there : job.n;
        chunks = (uint32_t)chunks_for(n);
        payload = offsets + chunks + 1;
        const uint64_t head = 256u + 4u * ((uint64_t)chunks + 1u);
        const uint64_t words = job.stream_bytes > head ? (job.stream_bytes - head) / 4u : 0u;
        payload_words = (uint32_t)(words < 0xffffffffu ? words : 0xffffffffu);
    }
    uint8_t* out = job.out;
    // One object, so that the order is the one written here: the table that every symbol is looked up in comes first,
    // at addresses small enough for the offset field of an LDS instruction (one addition less per symbol).
    struct Local {
        uint16_t  table[kTableEntries];                       // while it is being filled: ranks, one up
        LongCodes tables;
        uint32_t  in_wave[kThreads / 64][32];                 // [w][k]: symbols of length k among wave w's 64
        uint32_t  first_code[kThreads / 64][32];              // [w][k]: wave w's copy of: the first code of length k, from the 24th bit down
        uint32_t  first_rank[kThreads / 64][32];              // ... the place of its symbol by (length, symbol)
        uint16_t  entry_of_rank[256 + 2];                     // [rank + 1]; 0 at either end
        uint16_t  upto[kDecodeThreads];                       // the last rank in the table up to a thread's part, in its wave
        uint32_t  all_eight[4];                               // [w]: the codes of wave w's 64 symbols are eight bits long
        uint32_t  fitting;                                    // chunks of a pass whose slice fits the stage
        // the workgroup's slice of the payload, or the rings; four words lead in (a chunk's first window reads the one before it)
        __align__(16) uint32_t slice[4 + kStageWords + kChunkWordsMax + 8];
    };
    __shared__ Local local;
    LongCodes& tables = local.tables;
    uint32_t* const stage = local.slice + 4;
    const uint32_t s = threadIdx.x, wave = s >> 6, lane = s & 63u;
    uint32_t l = s < 256u ? len_in[s] : 0u;
    if (l > (uint32_t)kMaxLen) l = 0u;
    if (wave < 4u) {                                          // wave-uniform
        const uint64_t eight = __ballot(l == 8u);
        if (lane == 0) local.all_eight[wave] = eight == ~(uint64_t)0 ? 1u : 0u;
    }
    uint32_t* const table_words = reinterpret_cast<uint32_t*>(local.table);       // two entries each
    for (uint32_t i = s; i < (uint32_t)kTableEntries / 2u; i += kDecodeThreads) table_words[i] = 0u;
    if (s < kThreads / 64 * 32u) local.in_wave[s >> 5][s & 31u] = 0u;
    __syncthreads();
    const bool flat = (local.all_eight[0] & local.all_eight[1] & local.all_eight[2] & local.all_eight[3]) != 0u;
    uint32_t shift = 32u - kFastBits;
    int32_t add = 0;
    // Threads 0..255 stand for the 256 symbols: a symbol's place by (length, symbol), its code, and its rank written where
    // its part of the table starts; then every entry takes the last rank up to it, a scan over the workgroup, and the rank's
    // entry.  (Each entry by itself, its length from comparisons with all bounds and its symbol from that, was 7 us of the
    // 36 that a launch of few chunks took; this way it is 2.5.)
    const auto build_tables = [&] {
        uint32_t before = 0;                                  // symbols of this one's length before it in its wave
        if (wave < 4u) {                                      // wave-uniform
            const uint64_t same = lanes_alike(l);
            before = __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
            if (l && before == 0u) local.in_wave[wave][l] = (uint32_t)__popcll(same);
        }
        __syncthreads();
        // Lane k of every wave stands for length k.  The first code of length k is the sum over the shorter lengths j of their
        // symbols << (k - j); scaled by 2^(24 - k) that is a prefix sum (at most 2^31, whatever the lengths are).
        const bool a_length = lane >= 1u && lane <= (uint32_t)kMaxLen;
        const uint32_t of_length = a_length ? local.in_wave[0][lane & 31u] + local.in_wave[1][lane & 31u] + local.in_wave[2][lane & 31u] +
                                                  local.in_wave[3][lane & 31u] : 0u;
        const uint32_t scaled = a_length ? of_length << ((uint32_t)kMaxLen - lane) : 0u;
        const uint32_t codes_upto = wave_inclusive_scan(scaled), rank_upto = wave_inclusive_scan(of_length);
        const uint32_t first_code = codes_upto - scaled, first_rank = rank_upto - of_length;
        const uint32_t all_codes = last_lane(codes_upto);
        const uint64_t lengths = __ballot(of_length != 0u);
        const uint32_t longest = lengths ? 63u - (uint32_t)__builtin_clzll(lengths) : 0u;
        const uint32_t from = (uint32_t)__builtin_amdgcn_readlane((int)first_code, kFastBits + 1) >> (kMaxLen - kFastBits);
        uint32_t extra = 0;
        if (longest > (uint32_t)kFastBits && from < (1u << kFastBits)) {
            const uint32_t prefixes = (1u << kFastBits) - from;
            while (extra < longest - kFastBits && extra < kReach - kFastBits && from + (prefixes << (extra + 1u)) <= (uint32_t)kTableEntries) ++extra;
        }
        shift = 32u - kFastBits - extra;
        add = (int32_t)from - (int32_t)(from << extra);
        if (wave == 0 && a_length) {
            const uint64_t end = (uint64_t)codes_upto << (32 - kMaxLen);       // lengths no encoder wrote can claim more than there is
            tables.last[lane] = end > 0xffffffffull ? 0xffffffffu : end ? (uint32_t)end - 1u : 0u;
            tables.place[lane] = first_rank - (first_code >> ((uint32_t)kMaxLen - lane));
        }
        if (wave < 4u) {
            if (lane < 32u) {
                local.first_code[wave][lane] = first_code;
                local.first_rank[wave][lane] = first_rank;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // LDS operations of one wave complete in order
            if (l) {
                for (uint32_t w = 0; w < wave; ++w) before += local.in_wave[w][l];
                const uint32_t rank = (local.first_rank[wave][l] + before) & 0xffu;
                const uint32_t code = local.first_code[wave][l] + (before << ((uint32_t)kMaxLen - l));
                tables.sorted[rank] = (uint8_t)s;
                local.entry_of_rank[rank + 1u] = l <= kFastBits + extra ? (uint16_t)entry_of(s, l) : (uint16_t)0;
                // (codes longer than what an entry stands for may share one: none of them has an entry)
                if (code < (1u << kMaxLen)) local.table[table_index(shift, add, code << (32 - kMaxLen))] = (uint16_t)(rank + 1u);
            }
        } else if (s == 256u) {                               // and where the codes end
            local.entry_of_rank[0] = local.entry_of_rank[256 + 1] = (uint16_t)0;
            if (all_codes < (1u << kMaxLen)) local.table[table_index(shift, add, all_codes << (32 - kMaxLen))] = (uint16_t)(256u + 1u);
        }
        __syncthreads();
        constexpr int kWords = kTableEntries / 2 / kDecodeThreads;
        static_assert(kWords * 2 * kDecodeThreads == kTableEntries, "the threads share the table evenly");
        uint32_t two[kWords], upto = 0;
#pragma unroll
        for (int k = 0; k < kWords; ++k) {
            two[k] = table_words[s * kWords + k];
            upto = larger(upto, larger(two[k] & 0xffffu, two[k] >> 16));
        }
        local.upto[s] = (uint16_t)wave_inclusive_max(upto);
        __syncthreads();
        uint32_t rank = lane ? local.upto[s - 1u] : 0u;
        for (uint32_t w = 0; w < wave; ++w) rank = larger(rank, local.upto[64u * w + 63u]);
#pragma unroll
        for (int k = 0; k < kWords; ++k) {
            const uint32_t low = larger(rank, two[k] & 0xffffu);
            rank = larger(low, two[k] >> 16);
            table_words[s * kWords + k] = local.entry_of_rank[low] | (uint32_t)local.entry_of_rank[rank] << 16;
        }
        __syncthreads();
    };

    // The tables serve an equal share of the stream's chunks (a wave's worth at least), in passes of as many chunks as
    // there are threads at most.  The payload words of consecutive chunks are one contiguous slice.  A pass takes the
    // chunks whose slice fits the stage -- all there are threads for at up to 34.5 words per chunk on average (61 with 512
    // threads), fewer on streams that compress less, where the threads beyond sit the pass out -- brings the slice into LDS with contiguous loads, and
    // the threads read their words from there (a thread walking its chunk in memory would fetch a cache line per
    // word).  A pass that could seat few of its chunks, and offsets that do not describe a slice (no encoder wrote
    // them), go through per-thread rings instead.
    // Bytes that do not compress at all have codes of eight bits each, their own values: a copy with the bytes of each
    // word turned round.  (Decoded symbol by symbol, the chunks of 64 words each meet in one LDS bank.)
    if (flat) {                                       // workgroup-uniform
        const uint32_t each = (chunks + job.blocks - 1u) / job.blocks;
        const uint64_t stop = ((uint64_t)block + 1u) * each < chunks ? ((uint64_t)block + 1u) * each : chunks;
        for (uint64_t q = (uint64_t)block * each * 64u + threadIdx.x; q < stop * 64u; q += kDecodeThreads) {
            const uint32_t at = offsets[q >> 6] + (uint32_t)(q & 63u);
            const uint32_t word = at < payload_words ? payload[at] : 0u;
            if (4u * q + 4u <= n) {
                reinterpret_cast<uint32_t*>(out)[q] = __builtin_bswap32(word);
            } else {
                for (uint32_t k = 0; 4u * q + k < n; ++k) out[4u * q + k] = (uint8_t)(word >> (24u - 8u * k));
            }
        }
        return;
    }
    const uint32_t even = (chunks + job.blocks - 1u) / job.blocks;
    const uint64_t share = even < 64u ? 64u : even;
    const uint32_t chunk_stop = (uint32_t)((block + 1u) * share < chunks ? (block + 1u) * share : chunks);
    bool built = false;                                       // the tables: while the first slice is on its way
    for (uint32_t chunk0 = (uint32_t)(block * share < chunks ? block * share : chunks); chunk0 < chunk_stop;) {
        const uint32_t want = chunk_stop - chunk0 < (uint32_t)kDecodeThreads ? chunk_stop - chunk0 : (uint32_t)kDecodeThreads;
        const uint32_t slice_at = offsets[chunk0];
        // the chunks before the first whose end lies outside the stage (or the payload, or before the slice's start)
        const bool asked = threadIdx.x < want;
        const uint32_t my_end = asked ? offsets[chunk0 + threadIdx.x + 1u] : 0u;
        const bool fits = my_end >= slice_at && my_end - slice_at <= (uint32_t)kStageWords && my_end <= payload_words;
        if (threadIdx.x == 0) local.fitting = want;
        __syncthreads();
        {
            const uint64_t beyond = __ballot(asked && !fits);
            if (beyond && lane == 0) atomicMin(&local.fitting, wave * 64u + (uint32_t)__builtin_ctzll(beyond));
        }
        __syncthreads();
        const uint32_t fitting = local.fitting;
        // (workgroup-uniform) Below three quarters of its threads, of twelve waves at most, the rings do better: at some eight bits per
        // symbol chunks are 64 words long, the threads' words lie 64 apart in the stage and all in one LDS bank.
        const bool staged = fitting > 0u && 4u * fitting >= 3u * (want < 768u ? want : 768u);
        const uint32_t take = staged ? fitting : want;        // chunks of this pass
        const uint32_t slice_end = staged ? offsets[chunk0 + fitting] : slice_at;
        const uint32_t chunk = chunk0 + threadIdx.x;
        const bool live = threadIdx.x < take;
        const uint64_t base = (uint64_t)chunk * kChunk;
        const uint32_t valid = !live ? 0u : n - base < (uint64_t)kChunk ? (uint32_t)(n - base) : (uint32_t)kChunk;
        const uint32_t first_word = live ? offsets[chunk] : 0u;
        uint8_t* dst = out + base;
        // 16 bytes per load, nine loads of a thread in flight (twelve with 512 threads): one at a time, a slice of ~50 words
        // per thread would cost as many memory latencies.  The stage starts at the 16-byte boundary at or below the
        // slice's first word (`phase` words earlier); what the vectors cover beyond the payload's ends is
        // read as zero.
        const uint32_t slice_words = slice_end - slice_at;    // none where the pass is not staged
        const uint32_t phase = (uint32_t)(reinterpret_cast<uintptr_t>(payload + slice_at) >> 2) & 3u;
        const uint32_t vectors = staged ? (slice_words + phase + 3u) / 4u : 0u;
        constexpr int kVectors = kDecodeThreads > 512 ? 9 : 12;
        uint32_t v0 = 0;
        do {                                                  // workgroup-uniform
            u32x4 got[kVectors];
#pragma unroll
            for (int k = 0; k < kVectors; ++k) {
                const uint32_t v = v0 + k * kDecodeThreads + threadIdx.x;
                const int64_t w = (int64_t)slice_at + 4 * (int64_t)v - phase;  // below zero in the first vector at most
                const auto word_at = [&](int64_t g) { return g >= 0 && g < (int64_t)payload_words ? payload[g] : 0u; };
                got[k] = u32x4{0u, 0u, 0u, 0u};
                if (v < vectors) {
                    if (w >= 0 && w + 3 < (int64_t)payload_words) got[k] = *reinterpret_cast<const u32x4*>(payload + w);
                    else got[k] = u32x4{word_at(w), word_at(w + 1), word_at(w + 2), word_at(w + 3)};
                }
            }
            if (!built) build_tables();
            built = true;
#pragma unroll
            for (int k = 0; k < kVectors; ++k) {
                const uint32_t v = v0 + k * kDecodeThreads + threadIdx.x;
                if (v < vectors) *reinterpret_cast<u32x4*>(stage + 4u * v) = got[k];
            }
            v0 += (uint32_t)(kVectors * kDecodeThreads);
        } while (v0 < vectors);
        if (staged) {                                         // workgroup-uniform
            __syncthreads();
            // anything at all for a foreign stream: clamped, the reads stay inside the array (a chunk is at most 192 words)
            const uint32_t at = first_word - slice_at < slice_words ? first_word - slice_at : slice_words;
            const Lookup look{local.table, &tables, shift, add};
            if (shift != 32u - kFastBits) decode_chunk_staged<LINES, true>(valid, dst, look, stage + phase + at);      // wave-uniform
            else decode_chunk_staged<LINES, false>(valid, dst, look, stage + phase + at);
        } else if (live) {
            // a ring of eight words per thread: when four have been consumed, the four loaded at the
            // previous refill take their place and the next four are requested, so a load has the time
            // of four words' decoding to arrive
            uint32_t* mine = stage + threadIdx.x;             // word k of the ring at mine[(k & 7) * kDecodeThreads]
            uint32_t pending[4];
#pragma unroll
            for (int k = 0; k < 8; ++k) mine[k * kDecodeThreads] = first_word + k < payload_words ? payload[first_word + k] : 0u;
#pragma unroll
            for (int k = 0; k < 4; ++k) pending[k] = first_word + 8 + k < payload_words ? payload[first_word + 8 + k] : 0u;
            decode_chunk(valid, dst, Lookup{local.table, &tables, shift, add}, mine[0], [&](uint32_t taken) {
                if ((taken & 3u) == 0u) {                     // a block of four used up: refill the half of the ring just freed
                    const uint32_t slot = (taken + 4u) & 7u;
#pragma unroll
                    for (int k = 0; k < 4; ++k) mine[((slot + k) & 7u) * kDecodeThreads] = pending[k];
                    const uint32_t at = first_word + taken + 8u;
#pragma unroll
                    for (int k = 0; k < 4; ++k) pending[k] = at + k < payload_words ? payload[at + k] : 0u;
                }
                return mine[(taken & 7u) * kDecodeThreads];
            });
        }
        __syncthreads();                                      // the stage is the next pass's
        chunk0 += take;
    }
}

bool aligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }
uint64_t chunks_of(uint64_t n) { return (n + kChunk - 1) / kChunk; }
uint64_t groups_of(uint64_t n) { return (chunks_of(n) + kGroup - 1) / kGroup; }
constexpr uint64_t kMaxSymbols = ((uint64_t)1 << 32) - 1;

}  // namespace
}  // namespace fh

extern "C" {

size_t fh_huffman_stream_bytes(uint64_t n)
{
    if (n > fh::kMaxSymbols) return 0;
    return (size_t)(256u + 4u * (fh::chunks_of(n) + 1u) + 4u * (uint64_t)fh::kChunkWordsMax * fh::chunks_of(n));
}

size_t fh_huffman_workspace_bytes(uint64_t n)
{
    if (n > fh::kMaxSymbols) return 0;
    return (size_t)(4u * (256u + 256u + (fh::groups_of(n) > 0 ? fh::groups_of(n) : 1u)));
}

int32_t fh_huffman_batch_capacity(void) { return fh::kBatchStated; }

}  // extern "C"

namespace {

using namespace fh;

fh_status check_encode(const fh_huffman_encode_item& it)
{
    if (it.n > kMaxSymbols) return FH_ERR_BAD_NUMEL;
    if (!it.stream_out || !it.totals || !it.workspace || (it.n > 0 && !it.bytes)) return FH_ERR_NULL;
    if (!aligned(it.bytes, 16) || !aligned(it.stream_out, 16) || !aligned(it.totals, 8) || !aligned(it.workspace, 16) ||
        !aligned(it.n_device, 8))
        return FH_ERR_ALIGNMENT;
    if (it.stream_cap < fh_huffman_stream_bytes(it.n) || it.workspace_cap < fh_huffman_workspace_bytes(it.n))
        return FH_ERR_BUFFER_TOO_SMALL;
    return FH_OK;
}

fh_status check_decode(const fh_huffman_decode_item& it)
{
    if (it.n > kMaxSymbols) return FH_ERR_BAD_NUMEL;
    if (it.n == 0) return FH_OK;
    if (!it.stream_in || !it.out) return FH_ERR_NULL;
    if (!aligned(it.stream_in, 16) || !aligned(it.out, 16) || !aligned(it.n_device, 8)) return FH_ERR_ALIGNMENT;
    if (it.out_cap < it.n) return FH_ERR_BUFFER_TOO_SMALL;
    // not even the lengths and the offsets (with the count on the device: of the largest stream it may describe)
    if (it.stream_bytes < 256u + 4u * (chunks_of(it.n) + 1u)) return FH_ERR_BUFFER_TOO_SMALL;
    return FH_OK;
}

// The encoder's launches; `stored` null: there is no header to write to.
fh_status encode_all(const fh_huffman_encode_item* items, const StoredForm* stored, int32_t count, hipStream_t s)
{
    for (int32_t i = 0; i < count;) {
        // the same streams three times: a workgroup each | by histogram workgroups | by groups of chunks
        Batch<Stream> each, hist, grouped;
        reset(each); reset(hist); reset(grouped);
        while (i < count && each.count < kBatch) {
            const fh_huffman_encode_item& it = items[i];
            Stream lay;
            lay.chunks = (uint32_t)chunks_of(it.n);
            lay.groups = (uint32_t)groups_of(it.n);
            lay.out = static_cast<uint8_t*>(it.stream_out);
            lay.scratch = static_cast<uint32_t*>(it.workspace);
            lay.totals = static_cast<uint64_t*>(it.totals);
            lay.in = static_cast<const uint8_t*>(it.bytes);
            lay.n = it.n;
            lay.n_dev = static_cast<const uint64_t*>(it.n_device);
            lay.stored = stored ? stored[i] : StoredForm{nullptr, 0, 0};
            lay.hist_blocks = histogram_workgroups(it.n);
            if ((uint64_t)grouped.block_start[grouped.count] + lay.groups > (uint64_t)INT_MAX) {
                if (each.count == 0) return FH_ERR_BAD_NUMEL;
                break;
            }
            push(each, lay, 1);
            push(hist, lay, lay.hist_blocks);
            push(grouped, lay, lay.groups > 0 ? lay.groups : 1);       // one writes an empty stream's size
            ++i;
        }
        seal(each); seal(hist); seal(grouped);
        const dim3 streams((uint32_t)each.count), of_hist(hist.block_start[hist.count]), groups(grouped.block_start[grouped.count]);
        const bool scanned = group_sums_are_scanned(groups.x);
        if (of_hist.x > 0)
            with_arguments(hist, [&](const auto& args) { hipLaunchKernelGGL((huffman_histogram_kernel<FH_ARGS>), of_hist, dim3(kHistThreads), 0, s, args); });
        with_arguments(each, [&](const auto& args) { hipLaunchKernelGGL((huffman_code_kernel<FH_ARGS>), streams, dim3(kCodeThreads), 0, s, args); });
        with_arguments(grouped, [&](const auto& args) {
            hipLaunchKernelGGL((huffman_count_kernel<FH_ARGS>), groups, dim3(kGroupThreads), 0, s, args);
            if (!scanned) hipLaunchKernelGGL((huffman_write_kernel<false, FH_ARGS>), groups, dim3(kGroupThreads), 0, s, args);
        });
        if (scanned) {
            hipLaunchKernelGGL(huffman_scan_kernel, streams, dim3(kThreads), 0, s, each);
            hipLaunchKernelGGL((huffman_write_kernel<true, Batch<Stream>>), groups, dim3(kGroupThreads), 0, s, grouped);
        }
    }
    if (count == 0) return FH_OK;
    return hipGetLastError() == hipSuccess ? FH_OK : FH_ERR_LAUNCH;
}

}  // namespace

fh_status fh::huffman_encode_stored(const fh_huffman_encode_item* items, const StoredForm* stored, int32_t count, hipStream_t s)
{
    return encode_all(items, stored, count, s);
}

extern "C" {

fh_status fh_huffman_encode_batch(const fh_huffman_encode_item* items, int32_t count, void* stream)
{
    if (count < 0) return FH_ERR_BAD_COUNT;
    if (count > 0 && !items) return FH_ERR_NULL;
    for (int32_t i = 0; i < count; ++i) {                     // everything is checked before the first launch
        const fh_status st = check_encode(items[i]);
        if (st != FH_OK) return st;
    }
    return encode_all(items, nullptr, count, static_cast<hipStream_t>(stream));
}

fh_status fh_huffman_decode_batch(const fh_huffman_decode_item* items, int32_t count, void* stream)
{
    if (count < 0) return FH_ERR_BAD_COUNT;
    if (count > 0 && !items) return FH_ERR_NULL;
    for (int32_t i = 0; i < count; ++i) {
        const fh_status st = check_decode(items[i]);
        if (st != FH_OK) return st;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    // One workgroup per compute unit, each with an equal share of its stream's chunks.  A call whose chunks fit the
    // device in workgroups of 512 takes those, a wave per SIMD first (256 chunks); beyond that they would take two
    // passes, where the wide ones seat up to twice as many in one, and those get at least 512 chunks each, so that
    // every unit has one.  (A count that is on the device is an upper bound here: the index streams of the whole chain
    // come to some two thirds of it.  Where the count is exact, a workgroup's share is to fit its stage in one pass.)
    uint64_t narrow = 0, symbols = 0;
    for (int32_t i = 0; i < count; ++i) {
        const uint64_t seats = items[i].n_device ? (uint64_t)kDecodeThreadsSmall : kSmallSeats;
        narrow += (chunks_of(items[i].n) + seats - 1) / seats;
        symbols += items[i].n;
    }
    const bool small = narrow <= (uint64_t)kComputeUnits;
    const uint64_t per_group = small ? 256u : 512u;
    const uint64_t slots = kComputeUnits;                     // workgroups the device holds at once
    bool launched = false;
    for (int32_t i = 0; i < count;) {
        DecodeJob job[kBatch];
        uint64_t groups[kBatch], total = 0;
        int jobs = 0;
        for (; i < count && jobs < kBatch; ++i) {
            const fh_huffman_decode_item& it = items[i];
            if (it.n == 0) continue;                          // nothing to restore
            const uint64_t chunks = chunks_of(it.n);
            const uint64_t words = (it.stream_bytes - (256u + 4u * (chunks + 1u))) / 4u;
            DecodeJob& j = job[jobs];
            j.len = static_cast<const uint8_t*>(it.stream_in);
            j.offsets = reinterpret_cast<const uint32_t*>(j.len + 256);
            j.payload = j.offsets + chunks + 1;
            j.out = static_cast<uint8_t*>(it.out);
            j.n = it.n;
            j.n_dev = static_cast<const uint64_t*>(it.n_device);
            j.stream_bytes = it.stream_bytes;
            j.payload_words = (uint32_t)(words < 0xffffffffu ? words : 0xffffffffu);
            j.chunks = (uint32_t)chunks;
            groups[jobs] = (chunks + per_group - 1) / per_group;   // the decoder's own groups
            total += groups[jobs];
            ++jobs;
        }
        // A workgroup builds a stream's tables once and then decodes its share of the chunks.  With more groups
        // in the launch than workgroups fit on the device at once, every stream gets its share of that many
        // workgroups, and its chunks are dealt out evenly among them: all of them are resident from the start and
        // finish together (their last pass seats fewer chunks), whereas a launch of 1.4 times as many would run a
        // second, mostly empty round, and whole groups per workgroup would leave compute units without any.
        Batch<DecodeJob> b;
        reset(b);
        for (int k = 0; k < jobs; ++k) {
            uint64_t blocks = total <= slots ? groups[k] : groups[k] * slots / total;
            if (blocks < 1u) blocks = 1u;
            const uint64_t chunks = job[k].chunks;
            job[k].blocks = (uint32_t)(blocks < chunks ? blocks : chunks);
            if (!push(b, job[k], (int64_t)job[k].blocks)) return FH_ERR_BAD_NUMEL;   // cannot happen: a stream has at most 2^16 groups
        }
        seal(b);
        if (b.count > 0) {
            const dim3 grid(b.block_start[b.count]);
            if (!small && decode_in_whole_lines(symbols))
                hipLaunchKernelGGL((huffman_decode_kernel<kDecodeThreads, true, Batch<DecodeJob>>), grid, dim3(kDecodeThreads), 0, s, b);
            else with_arguments(b, [&](const auto& args) {
                if (small) hipLaunchKernelGGL((huffman_decode_kernel<kDecodeThreadsSmall, false, FH_ARGS>), grid, dim3(kDecodeThreadsSmall), 0, s, args);
                else hipLaunchKernelGGL((huffman_decode_kernel<kDecodeThreads, false, FH_ARGS>), grid, dim3(kDecodeThreads), 0, s, args);
            });
            launched = true;
        }
    }
    if (!launched) return FH_OK;
    return hipGetLastError() == hipSuccess ? FH_OK : FH_ERR_LAUNCH;
}

fh_status fh_huffman_encode(const void* bytes, uint64_t n, void* stream_out, size_t stream_cap, void* totals,
                            void* workspace, size_t workspace_cap, void* stream)
{
    fh_huffman_encode_item it;
    it.n_device = nullptr;
    it.bytes = bytes; it.n = n; it.stream_out = stream_out; it.stream_cap = stream_cap; it.totals = totals;
    it.workspace = workspace; it.workspace_cap = workspace_cap;
    return fh_huffman_encode_batch(&it, 1, stream);
}

fh_status fh_huffman_decode(const void* stream_in, size_t stream_bytes, uint64_t n, void* out, size_t out_cap,
                            void* stream)
{
    fh_huffman_decode_item it;
    it.n_device = nullptr;
    it.stream_in = stream_in; it.stream_bytes = stream_bytes; it.n = n; it.out = out; it.out_cap = out_cap;
    return fh_huffman_decode_batch(&it, 1, stream);
}

}  // extern "C"
