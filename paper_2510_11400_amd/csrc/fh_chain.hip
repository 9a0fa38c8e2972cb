// The channel-wise mix compressor as one call each way (paper Section 4.4.1 from its first
// sentence to its last; Algorithm 1 sees exactly these two actions, compress and decompress):
//
//   forward   classify channels (three-sigma rule) -> number the salient ones -> quantise the
//             normal channels, salient ones to a raw store -> the raw store's feature maps as
//             sparse blocks (CSR) and dense blocks (Lorenzo prediction within an error bound)
//             -> Huffman coding of the index stream;
//   backward  Huffman decoding -> maps rebuilt -> normal channels dequantised, salient channels
//             taken from the maps.
//
// Every stage is the library's own batched call; this file only lays the caller's two buffers
// out, strings the calls together on one stream, and adds two small kernels: one that takes the
// masks from the outlier counts, numbers the salient channels of every tensor of the call, clears
// the headers and, where the sparse stage does not, the rows of the raw stores that no channel uses (they read as zero), and one
// that adds up what a tensor's stored form occupies where the entropy stage does not do that.  Sizes that depend on the data (stream lengths) never visit the host:
// the sparse stage's totals feed the Huffman stage through device memory.
#include "../../include/fedhybrid.h"

#include "fh_batch.hpp"
#include "fh_rules.hpp"
#include "fh_scan.hpp"
#include "fh_stages.hpp"

#include <vector>

namespace fh {
namespace {

constexpr int kPrepThreads = 1024;
constexpr int kSlotPerThread = 16;                 // 1024 * 16 = the largest channel count
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct PrepItem {
    const uint32_t* counts;                        // outliers per channel
    int64_t         min_outliers;
    uint8_t*        mask;
    int16_t*        slots;
    uint64_t*       header;                        // 8 words, cleared; [7] = slots in use
    uint8_t*        raw;                           // the raw store: [outer][raw_channels][row_bytes]
    uint64_t        row_bytes;
    uint32_t        outer;                         // samples whose unused rows are to be cleared
    int32_t         channels, raw_channels;
    uint32_t        blocks;                        // workgroups of this item
};
constexpr uint32_t kClearUnit = 16384;             // bytes that a wave clears at a time
constexpr uint32_t kWholeBelow = 4096;             // bytes of a sample's rows below which the raw store is cleared whole

// `bytes` bytes at p (element-aligned, 2 or 4) by one wave
__device__ __forceinline__ void clear_bytes(uint8_t* p, uint64_t bytes, uint32_t lane)
{
    const u32x4 zero = {0u, 0u, 0u, 0u};
    const uint64_t lead = (16u - (reinterpret_cast<uintptr_t>(p) & 15u)) & 15u, head = lead < bytes ? lead : bytes;
    const uint64_t vectors = (bytes - head) / 16u, tail = head + vectors * 16u;
    if (2u * lane < head) *reinterpret_cast<uint16_t*>(p + 2u * lane) = 0u;
    for (uint64_t v = lane; v < vectors; v += 64u) reinterpret_cast<u32x4*>(p + head)[v] = zero;
    if (tail + 2u * lane < bytes) *reinterpret_cast<uint16_t*>(p + tail + 2u * lane) = 0u;
}

// Workgroup 0 of an item: mask[c] = channel c has min_outliers outliers or more, slots[c] = number
// of salient channels before c while that is below raw_channels, -1 for every other channel (each
// thread owns 16 consecutive channels, the per-thread counts are scanned over the workgroup), and the
// header cleared.  All workgroups of the item: the raw store's rows that no
// channel uses cleared.  (The rows in use are written whole by the quantiser: with 4 % of the channels salient and room
// for a sixteenth, clearing them as well wrote 36 MB instead of 13 MB for the MobileNetV2-style set, 13 us against 8.6.)
template <typename Args>
__global__ __launch_bounds__(kPrepThreads) void chain_prepare_kernel(const Args batch)
{
    uint32_t block;
    const PrepItem& it = item_of(batch, blockIdx.x, block);
    __shared__ uint32_t of_wave[kPrepThreads / 64];
    const int t = threadIdx.x;
    const uint32_t wave_here = (uint32_t)__builtin_amdgcn_readfirstlane(t >> 6);
    const int first = t * kSlotPerThread;
    uint32_t salient = 0;                                     // bit k: channel first + k
    for (int k = 0; k < kSlotPerThread; ++k) {
        const int c = first + k;
        if (c < it.channels && (int64_t)it.counts[c] >= it.min_outliers) salient |= 1u << k;
    }
    const uint32_t mine = (uint32_t)__popc(salient), upto = wave_inclusive_scan(mine);
    if ((t & 63) == 63) of_wave[wave_here] = upto;
    __syncthreads();
    uint32_t all = 0, before = upto - mine;                   // salient channels; those before this thread's first
    for (uint32_t w = 0; w < (uint32_t)(kPrepThreads / 64); ++w) {
        if (w < wave_here) before += of_wave[w];
        all += of_wave[w];
    }
    const uint32_t used = all < (uint32_t)it.raw_channels ? all : (uint32_t)it.raw_channels;
    if (block == 0) {                                         // workgroup-uniform
        int rank = (int)before;
        for (int k = 0; k < kSlotPerThread; ++k) {
            const int c = first + k;
            if (c >= it.channels) break;
            const bool is = (salient >> k) & 1u;
            it.mask[c] = is ? 1u : 0u;
            it.slots[c] = (int16_t)(is && rank < it.raw_channels ? rank : -1);
            if (is) ++rank;
        }
        if (t < 7) it.header[t] = 0u;
        if (t == 7) it.header[7] = used;
    }
    // The unused rows of a sample are one piece; a wave takes a part of one at a time.  Pieces of a few hundred bytes
    // ([tokens][hidden] tensors) are cleared together with what lies between them: one by one they took 56 us for
    // the 24 tensors of an encoder, whole 13 us, and as the 16-byte vectors that have a part in an unused row 12.
    const uint64_t sample = (uint64_t)it.raw_channels * it.row_bytes, unused = (uint64_t)(it.raw_channels - (int)used) * it.row_bytes;
    const bool whole = sample < kWholeBelow;
    const uint64_t samples = whole ? 1u : it.outer, piece = whole ? (used < (uint32_t)it.raw_channels ? it.outer * sample : 0u) : unused;
    uint8_t* const clear = whole ? it.raw : it.raw + (uint64_t)used * it.row_bytes;
    const uint32_t parts = (uint32_t)((piece + kClearUnit - 1u) / kClearUnit), waves = it.blocks * (kPrepThreads / 64);
    const uint32_t wave = block * (kPrepThreads / 64) + wave_here;
    const uint64_t units = samples * parts;
    for (uint64_t u = wave; u < units; u += waves) {          // wave-uniform
        const uint64_t o = u / parts, at = (u - o * parts) * kClearUnit;
        clear_bytes(clear + o * sample + at, piece - at < kClearUnit ? piece - at : kClearUnit, (uint32_t)t & 63u);
    }
}

struct SummaryItem {
    uint64_t* header;
    uint64_t  fixed_bytes;                         // header + slots + codes + meta + info
    uint32_t  value_size;                          // bytes per element of the value stream
};
struct SummaryBatch { int32_t count; SummaryItem item[kBatch]; };

__global__ void chain_summary_kernel(const SummaryBatch batch)
{
    const int i = threadIdx.x;
    if (i >= batch.count) return;
    const SummaryItem& it = batch.item[i];
    it.header[6] = it.fixed_bytes + it.header[0] * it.value_size + it.header[1];
}

size_t up(size_t v) { return (v + 255u) & ~(size_t)255u; }
size_t elem_size(int dtype) { return dtype == FH_F32 ? 4u : 2u; }
bool aligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

// Everything about an item that does not involve its buffers.
fh_status check_shape(const fh_mix_item& it, int64_t* numel)
{
    if (it.x_dtype != FH_F32 && it.x_dtype != FH_BF16) return FH_ERR_BAD_DTYPE;
    if (it.reserved != 0 || it.quant.reserved != 0) return FH_ERR_BAD_PARAM;
    if (it.quant.group_size != 64 && it.quant.group_size != 128 && it.quant.group_size != 256) return FH_ERR_BAD_GROUP;
    if (it.quant.bits != 2 && it.quant.bits != 4 && it.quant.bits != 8) return FH_ERR_BAD_BITS;
    if (it.quant.rounding != FH_ROUND_NEAREST && it.quant.rounding != FH_ROUND_STOCHASTIC) return FH_ERR_BAD_ROUND;
    if (it.outer < 0 || it.channels < 1 || it.channels > 16384 || it.inner < 1) return FH_ERR_BAD_SHAPE;
    if (it.raw_channels < 0 || it.raw_channels > it.channels) return FH_ERR_BAD_SHAPE;
    if (!(it.k_sigma > 0.0) || it.min_outliers < 1) return FH_ERR_BAD_PARAM;
    if (it.entropy != 0 && it.entropy != 1) return FH_ERR_BAD_PARAM;
    const int64_t limit = (int64_t)1 << 31;                   // the routed quantiser indexes elements with 32 bits
    if (it.inner > limit || it.channels * it.inner > limit) return FH_ERR_BAD_NUMEL;
    if (it.outer > limit / (it.channels * it.inner)) return FH_ERR_BAD_NUMEL;
    *numel = it.outer * it.channels * it.inner;
    const int64_t kept = it.outer * it.raw_channels * it.inner;
    if (kept > 0) {
        if (it.window != 2 && it.window != 4 && it.window != 8) return FH_ERR_BAD_PARAM;
        if (it.maps < 1 || it.h < 1 || it.w < 1) return FH_ERR_BAD_SHAPE;
        if (it.h > kept || it.w > kept / it.h || it.maps != kept / (it.h * it.w) || it.maps * it.h * it.w != kept)
            return FH_ERR_BAD_SHAPE;                          // the maps must be exactly the raw store
    }
    return FH_OK;
}

fh_status layout_of(const fh_mix_item& it, fh_mix_regions* r)
{
    int64_t numel = 0;
    const fh_status st = check_shape(it, &numel);
    if (st != FH_OK) return st;
    *r = fh_mix_regions{};
    const int64_t kept = it.outer * it.raw_channels * it.inner;
    r->packed_bytes = fh_packed_bytes(numel, it.quant.bits);
    r->meta_bytes = fh_meta_bytes(numel, it.quant.group_size);
    r->slots_bytes = 2u * (size_t)it.channels;
    r->raw_bytes = (size_t)kept * elem_size(it.x_dtype);
    r->classify_ws_bytes = fh_classify_workspace_bytes(numel);
    if (kept > 0) {
        r->info_bytes = fh_sparse_info_bytes(it.maps, it.h, it.w, it.window);
        r->values_cap = r->raw_bytes;
        r->indices_cap = fh_sparse_index_bytes(it.maps, it.h, it.w, it.window);
        r->sparse_ws_bytes = fh_sparse_workspace_bytes(it.maps, it.h, it.w, it.window);
        if (r->indices_cap >= ((size_t)1 << 32)) return FH_ERR_BAD_NUMEL;
        if (it.entropy) {
            r->huffman_cap = fh_huffman_stream_bytes(r->indices_cap);
            r->huffman_ws_bytes = fh_huffman_workspace_bytes(r->indices_cap);
        }
    }
    size_t at = 0;
    const auto place = [&at](size_t bytes) { const size_t here = at; at += up(bytes); return here; };
    r->header = place(64);
    r->slots = place(r->slots_bytes);
    r->packed = place(r->packed_bytes);
    r->meta = place(r->meta_bytes);
    r->info = place(r->info_bytes);
    r->values = place(r->values_cap);
    r->indices = it.entropy ? 0 : place(r->indices_cap);
    r->huffman = it.entropy ? place(r->huffman_cap) : 0;
    r->store_bytes = at;
    at = 0;
    r->stats = place(32);
    r->counts = place(4u * (size_t)it.channels);
    r->mask = place((size_t)it.channels);
    r->classify_ws = place(r->classify_ws_bytes);
    r->raw = place(r->raw_bytes);
    r->sparse_ws = place(r->sparse_ws_bytes);
    r->indices_ws = it.entropy ? place(r->indices_cap) : 0;
    r->huffman_ws = place(r->huffman_ws_bytes);
    r->workspace_bytes = at;
    return FH_OK;
}

fh_status check_item(const fh_mix_item& it, bool forward, fh_mix_regions* r, int64_t* numel)
{
    fh_status st = layout_of(it, r);
    if (st != FH_OK) return st;
    check_shape(it, numel);
    if (!forward && it.out_dtype != FH_F32 && it.out_dtype != FH_BF16) return FH_ERR_BAD_DTYPE;
    if (!it.store || !it.workspace) return FH_ERR_NULL;
    if (*numel > 0 && (forward ? !it.x : !it.out)) return FH_ERR_NULL;
    if (!aligned(it.store, 256) || !aligned(it.workspace, 256) || !aligned(forward ? it.x : it.out, 16)) return FH_ERR_ALIGNMENT;
    if (it.store_cap < r->store_bytes || it.workspace_cap < r->workspace_bytes) return FH_ERR_BUFFER_TOO_SMALL;
    if (!forward && it.out_cap < (size_t)*numel * elem_size(it.out_dtype)) return FH_ERR_BUFFER_TOO_SMALL;
    return FH_OK;
}

uint8_t* at(void* base, size_t off) { return static_cast<uint8_t*>(base) + off; }

// Which maps of an item's raw store hold anything.  Where a map is a row of the store, the sparse encoder is told, and does not read the
// others but sets them to zero; where it is not ([tokens][hidden] tensors), or an empty tile would not be a sparse one, those
// rows are cleared before it reads them.
MapsInUse rows_in_use(const fh_mix_item& it, const fh_mix_regions& reg)
{
    const bool by_rows = it.h * it.w == it.inner && it.tau >= 0.0f;
    return by_rows ? maps_in_use(reinterpret_cast<const uint64_t*>(at(it.store, reg.header)) + 7, (uint32_t)it.raw_channels)
                   : MapsInUse{nullptr, 1, 0};
}

}  // namespace
}  // namespace fh

extern "C" {

fh_status fh_mix_layout(const fh_mix_item* item, fh_mix_regions* regions)
{
    if (!item || !regions) return FH_ERR_NULL;
    return fh::layout_of(*item, regions);
}

fh_status fh_mix_compress_batch(const fh_mix_item* items, int32_t count, void* stream)
{
    using namespace fh;
    if (count < 0) return FH_ERR_BAD_COUNT;
    if (count > 0 && !items) return FH_ERR_NULL;
    std::vector<fh_mix_regions> reg((size_t)count);
    std::vector<int64_t> numel((size_t)count);
    for (int32_t i = 0; i < count; ++i) {                     // everything is checked before the first launch
        const fh_status st = check_item(items[i], true, &reg[i], &numel[i]);
        if (st != FH_OK) return st;
    }
    if (count == 0) return FH_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    fh_status st;

    // 1. three-sigma statistics, outlier counts, salient mask
    std::vector<fh_classify_item> cls((size_t)count);
    std::vector<uint32_t*> ranges((size_t)count);
    for (int32_t i = 0; i < count; ++i) {
        const fh_mix_item& it = items[i];
        fh_classify_item& c = cls[i];
        c = fh_classify_item{};
        c.x = it.x; c.x_dtype = it.x_dtype;
        c.outer = it.outer; c.channels = it.channels; c.inner = it.inner;
        c.k_sigma = it.k_sigma; c.min_outliers = it.min_outliers;
        c.workspace = at(it.workspace, reg[i].classify_ws); c.workspace_cap = reg[i].classify_ws_bytes;
        c.stats = at(it.workspace, reg[i].stats); c.counts = at(it.workspace, reg[i].counts);
        c.mask = at(it.workspace, reg[i].mask);
    }
    // What the quantiser will be given (step 3, or partly before step 1).
    std::vector<fh_mixed_item> mix((size_t)count);
    for (int32_t i = 0; i < count; ++i) {
        const fh_mix_item& it = items[i];
        fh_mixed_item& m = mix[i];
        m = fh_mixed_item{};
        m.x = it.x; m.x_dtype = it.x_dtype; m.out_dtype = FH_F32;
        m.outer = it.outer; m.channels = it.channels; m.inner = it.inner;
        m.slots = at(it.store, reg[i].slots); m.raw_channels = it.raw_channels;
        m.packed = at(it.store, reg[i].packed); m.packed_cap = reg[i].packed_bytes;
        m.meta = at(it.store, reg[i].meta); m.meta_cap = reg[i].meta_bytes;
        m.raw = at(it.workspace, reg[i].raw); m.raw_cap = reg[i].raw_bytes; m.raw_dtype = it.x_dtype;
        m.params = it.quant;
        m.rows_in_use = at(it.store, reg[i].header) + 7 * sizeof(uint64_t);
    }
    // Where few spans can hold kept elements, the tensors are quantised as if nothing were kept while the
    // classification's first pass reads them, and step 3 does those spans again: one read of the tensors less.
    // On the MobileNetV2-style set that is a ninth of the spans at most: 112 us and 24 us for the two steps, where the
    // first pass by itself and the routed quantiser take 87 us and 121 us.  Not where every span holds kept elements ([tokens][hidden]) or a quarter of them may.
    // The value ranges lie in memory that is written whole after the classification: the raw store's where the
    // codes are there already, the codes' otherwise.
    bool first = true;
    double elements = 0.0, again = 0.0;
    for (int32_t i = 0; i < count; ++i) {
        first = first && (numel[i] == 0 || (items[i].inner > 1 && reg[i].raw_bytes >= range_bytes(numel[i])));
        elements += (double)numel[i];
        again += (double)items[i].outer * (double)items[i].raw_channels * (double)(items[i].inner + 2 * kFirstSpan);
    }
    first = first && 4.0 * again <= elements;
    for (int32_t i = 0; i < count; ++i) {
        void* const place = first ? at(items[i].workspace, reg[i].raw) : at(items[i].store, reg[i].packed);
        const size_t room = first ? reg[i].raw_bytes : reg[i].packed_bytes;
        ranges[i] = room >= range_bytes(numel[i]) ? static_cast<uint32_t*>(place) : nullptr;
    }
    if (first && (st = compress_first(mix.data(), cls.data(), ranges.data(), count, s)) != FH_OK) return st;
    if ((st = classify_counts(cls.data(), ranges.data(), count, first, s)) != FH_OK) return st;

    // 2. masks from the counts, slots from the masks; headers and the raw stores' unused rows cleared
    for (int32_t i = 0; i < count;) {
        Batch<PrepItem> b;
        reset(b);
        for (; i < count && b.count < kBatch; ++i) {
            const fh_mix_item& it = items[i];
            PrepItem p;
            p.counts = reinterpret_cast<const uint32_t*>(at(it.workspace, reg[i].counts));
            p.min_outliers = it.min_outliers;
            p.mask = at(it.workspace, reg[i].mask);
            p.slots = reinterpret_cast<int16_t*>(at(it.store, reg[i].slots));
            p.header = reinterpret_cast<uint64_t*>(at(it.store, reg[i].header));
            p.raw = at(it.workspace, reg[i].raw);
            p.row_bytes = (uint64_t)it.inner * elem_size(it.x_dtype);
            p.outer = reg[i].raw_bytes && !rows_in_use(it, reg[i]).count ? (uint32_t)it.outer : 0u;
            p.channels = (int32_t)it.channels;
            p.raw_channels = (int32_t)it.raw_channels;
            // every workgroup counts the salient channels first: 16 KiB of rows for each of its waves at least
            const uint64_t want = p.outer ? reg[i].raw_bytes / ((kPrepThreads / 64) * kClearUnit) + 1u : 1u;
            p.blocks = (uint32_t)(want < 512u ? want : 512u);
            push(b, p, p.blocks);
        }
        seal(b);
        const dim3 grid(b.block_start[b.count]);
        with_arguments(b, [&](const auto& args) { hipLaunchKernelGGL((chain_prepare_kernel<FH_ARGS>), grid, dim3(kPrepThreads), 0, s, args); });
    }

    // 3. normal channels quantised, salient channels to the raw store
    if ((st = first ? compress_kept(mix.data(), count, s) : fh_compress_mixed_batch(mix.data(), count, stream)) != FH_OK) return st;

    // 4. the raw stores as sparse / predicted blocks; 5. their index streams Huffman-coded
    std::vector<fh_sparse_encode_item> sp;
    std::vector<MapsInUse> use;
    std::vector<fh_huffman_encode_item> hf;
    std::vector<StoredForm> stored;
    const auto fixed_bytes = [&](int32_t i) {                 // of the stored form: header, codes, meta, slots and info bytes
        return 64u + reg[i].packed_bytes + reg[i].meta_bytes + (reg[i].raw_bytes ? reg[i].slots_bytes + reg[i].info_bytes : 0u);
    };
    for (int32_t i = 0; i < count; ++i) {
        const fh_mix_item& it = items[i];
        if (reg[i].raw_bytes == 0) continue;
        uint64_t* header = reinterpret_cast<uint64_t*>(at(it.store, reg[i].header));
        fh_sparse_encode_item e = {};
        e.x = at(it.workspace, reg[i].raw); e.dtype = it.x_dtype; e.n = it.window;
        e.maps = it.maps; e.h = it.h; e.w = it.w; e.tau = it.tau; e.eps = it.eps;
        e.info = at(it.store, reg[i].info); e.info_cap = reg[i].info_bytes;
        e.values = at(it.store, reg[i].values); e.values_cap = reg[i].values_cap;
        e.indices = it.entropy ? at(it.workspace, reg[i].indices_ws) : at(it.store, reg[i].indices);
        e.indices_cap = reg[i].indices_cap;
        e.totals = header;
        e.workspace = at(it.workspace, reg[i].sparse_ws); e.workspace_cap = reg[i].sparse_ws_bytes;
        sp.push_back(e);
        use.push_back(rows_in_use(it, reg[i]));
        if (it.entropy) {
            fh_huffman_encode_item h = {};
            h.bytes = e.indices; h.n = reg[i].indices_cap; h.n_device = header + 1;
            h.stream_out = at(it.store, reg[i].huffman); h.stream_cap = reg[i].huffman_cap;
            h.totals = header + 4;
            h.workspace = at(it.workspace, reg[i].huffman_ws); h.workspace_cap = reg[i].huffman_ws_bytes;
            hf.push_back(h);
            stored.push_back(StoredForm{header, fixed_bytes(i), (uint32_t)elem_size(it.x_dtype)});
        }
    }
    if (!sp.empty() && (st = sparse_encode_rows(sp.data(), use.data(), (int32_t)sp.size(), s)) != FH_OK) return st;
    if (!hf.empty() && (st = huffman_encode_stored(hf.data(), stored.data(), (int32_t)hf.size(), s)) != FH_OK) return st;

    // 6. what each stored form occupies, where the entropy stage has not said so
    for (int32_t i = 0; i < count;) {
        SummaryBatch b;
        b.count = 0;
        for (; i < count && b.count < kBatch; ++i) {
            if (reg[i].raw_bytes && items[i].entropy) continue;
            SummaryItem& q = b.item[b.count++];
            q.header = reinterpret_cast<uint64_t*>(at(items[i].store, reg[i].header));
            q.fixed_bytes = fixed_bytes(i);
            q.value_size = (uint32_t)elem_size(items[i].x_dtype);
        }
        if (b.count > 0) hipLaunchKernelGGL(chain_summary_kernel, dim3(1), dim3(64), 0, s, b);
    }
    return hipGetLastError() == hipSuccess ? FH_OK : FH_ERR_LAUNCH;
}

fh_status fh_mix_decompress_batch(const fh_mix_item* items, int32_t count, void* stream)
{
    using namespace fh;
    if (count < 0) return FH_ERR_BAD_COUNT;
    if (count > 0 && !items) return FH_ERR_NULL;
    std::vector<fh_mix_regions> reg((size_t)count);
    std::vector<int64_t> numel((size_t)count);
    for (int32_t i = 0; i < count; ++i) {
        const fh_status st = check_item(items[i], false, &reg[i], &numel[i]);
        if (st != FH_OK) return st;
    }
    if (count == 0) return FH_OK;
    fh_status st;

    // the index streams back, then the maps (the raw stores), then the tensors
    std::vector<fh_huffman_decode_item> hf;
    std::vector<fh_sparse_decode_item> sp;
    for (int32_t i = 0; i < count; ++i) {
        const fh_mix_item& it = items[i];
        if (reg[i].raw_bytes == 0) continue;
        const uint64_t* header = reinterpret_cast<const uint64_t*>(at(it.store, reg[i].header));
        const void* indices = it.entropy ? at(it.workspace, reg[i].indices_ws) : at(it.store, reg[i].indices);
        if (it.entropy) {
            fh_huffman_decode_item h = {};
            h.stream_in = at(it.store, reg[i].huffman); h.stream_bytes = reg[i].huffman_cap;
            h.n = reg[i].indices_cap; h.n_device = header + 1;
            h.out = at(it.workspace, reg[i].indices_ws); h.out_cap = reg[i].indices_cap;
            hf.push_back(h);
        }
        fh_sparse_decode_item d = {};
        d.info = at(it.store, reg[i].info);
        d.values = at(it.store, reg[i].values); d.values_bytes = reg[i].values_cap;
        d.indices = indices; d.indices_bytes = reg[i].indices_cap;
        d.dtype = it.x_dtype; d.n = it.window; d.maps = it.maps; d.h = it.h; d.w = it.w; d.eps = it.eps;
        d.out = at(it.workspace, reg[i].raw); d.out_cap = reg[i].raw_bytes;
        d.workspace = at(it.workspace, reg[i].sparse_ws); d.workspace_cap = reg[i].sparse_ws_bytes;
        sp.push_back(d);
    }
    if (!hf.empty() && (st = fh_huffman_decode_batch(hf.data(), (int32_t)hf.size(), stream)) != FH_OK) return st;
    uint64_t map_bytes = 0;
    for (const fh_sparse_decode_item& d : sp) map_bytes += d.out_cap;
    if (!sp.empty()) {
        st = maps_stay_in_cache(map_bytes) ? sparse_decode_for_next(sp.data(), (int32_t)sp.size(), static_cast<hipStream_t>(stream))
                                           : fh_sparse_decode_batch(sp.data(), (int32_t)sp.size(), stream);
        if (st != FH_OK) return st;
    }

    std::vector<fh_mixed_item> mix((size_t)count);
    for (int32_t i = 0; i < count; ++i) {
        const fh_mix_item& it = items[i];
        fh_mixed_item& m = mix[i];
        m = fh_mixed_item{};
        m.x_dtype = FH_F32; m.out_dtype = it.out_dtype;
        m.outer = it.outer; m.channels = it.channels; m.inner = it.inner;
        m.slots = at(it.store, reg[i].slots); m.raw_channels = it.raw_channels;
        m.packed = at(it.store, reg[i].packed); m.packed_cap = reg[i].packed_bytes;
        m.meta = at(it.store, reg[i].meta); m.meta_cap = reg[i].meta_bytes;
        m.raw = at(it.workspace, reg[i].raw); m.raw_cap = reg[i].raw_bytes; m.raw_dtype = it.x_dtype;
        m.out = it.out; m.out_cap = it.out_cap;
        m.params = it.quant;
        m.rows_in_use = at(it.store, reg[i].header) + 7 * sizeof(uint64_t);
    }
    return fh_decompress_mixed_batch(mix.data(), count, stream);
}

fh_status fh_mix_compress(const fh_mix_item* item, void* stream)
{
    return item ? fh_mix_compress_batch(item, 1, stream) : FH_ERR_NULL;
}

fh_status fh_mix_decompress(const fh_mix_item* item, void* stream)
{
    return item ? fh_mix_decompress_batch(item, 1, stream) : FH_ERR_NULL;
}

}  // extern "C"
