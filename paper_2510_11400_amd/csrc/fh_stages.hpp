// What the whole-chain call needs of the stages beyond their public entry points: the same calls with small pieces of
// work left out that a kernel of the chain does on its way, and with scratch given separately.  The items of all
// calls have been checked.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <hip/hip_runtime.h>

#include "../../include/fedhybrid.h"

namespace fh {

// Bytes of a tensor's value ranges: one word per 128 elements of its 1024-element spans.
inline size_t range_bytes(int64_t numel) { return numel > 0 ? (size_t)((numel + 1023) / 1024) * 32u : 0u; }

// fh_classify_channels_batch without the masks (which follow from the counts), and with ranges[i] (16-byte aligned,
// range_bytes() of item i, or null: the count pass then reads the whole tensor).  `first_pass_done`: the partial sums
// and the ranges (all given) are there.
fh_status classify_counts(const fh_classify_item* items, uint32_t* const* ranges, int32_t count, bool first_pass_done,
                          hipStream_t s);

// What the classification adds to, cleared by its first pass.
struct Cleared { uint32_t* counts; uint8_t* mask; int32_t channels; };
inline Cleared cleared_of(const fh_classify_item& it)
{
    return Cleared{static_cast<uint32_t*>(it.counts), static_cast<uint8_t*>(it.mask), (int32_t)it.channels};
}

// The forward side in two steps, for tensors of which few elements are kept: compress_first quantises the tensors as if
// nothing were kept and makes the classification's first pass on the way (partial sums at classify[i].workspace, ranges
// at ranges[i]); compress_kept, once the slots are known, does fh_compress_mixed_batch's work for the spans of the
// tensors that hold kept elements.  Together they leave what fh_compress_mixed_batch leaves.
fh_status compress_first(const fh_mixed_item* items, const fh_classify_item* classify, uint32_t* const* ranges, int32_t count,
                         hipStream_t s);
fh_status compress_kept(const fh_mixed_item* items, int32_t count, hipStream_t s);
constexpr int64_t kFirstSpan = 2048;               // elements of such a span at most

// Maps that are the rows of a raw store, `rows` to a sample, of which the first *count (device) are in use: the others are
// not read, count as zeros and are set to zero.  scale: floor(2^32 / rows), all ones for a single row.  count null: all maps are in use.
struct MapsInUse { const uint64_t* count; uint32_t rows, scale; };
inline MapsInUse maps_in_use(const uint64_t* count, uint32_t rows)
{
    return MapsInUse{count, rows, rows > 1u ? (uint32_t)(((uint64_t)1 << 32) / rows) : 0xffffffffu};
}
// fh_sparse_encode_batch with use[i] of item i (whose tau is not below 0).
fh_status sparse_encode_rows(const fh_sparse_encode_item* items, const MapsInUse* use, int32_t count, hipStream_t s);
// fh_sparse_decode_batch for maps that the next kernel on the stream finds in the caches (maps_stay_in_cache).
fh_status sparse_decode_for_next(const fh_sparse_decode_item* items, int32_t count, hipStream_t s);

// fh_huffman_encode_batch with the bytes that the stored form of the tensor occupies written to header[6] on the way:
// fixed_bytes + header[0] * value_size + the stream's bytes.
struct StoredForm { uint64_t* header; uint64_t fixed_bytes; uint32_t value_size; };
fh_status huffman_encode_stored(const fh_huffman_encode_item* items, const StoredForm* stored, int32_t count, hipStream_t s);

}  // namespace fh
