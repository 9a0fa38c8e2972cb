// What the whole-chain call needs of the classification beyond the public entry points: the same call with a place
// for the value ranges of each tensor given separately, so that it can lie in memory that is free at that time.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <hip/hip_runtime.h>

#include "../../include/fedhybrid.h"

namespace fh {

// Bytes of a tensor's value ranges: one word per 128 elements of its 1024-element spans.
inline size_t range_bytes(int64_t numel) { return numel > 0 ? (size_t)((numel + 1023) / 1024) * 32u : 0u; }

// fh_classify_channels_batch with ranges[i] (16-byte aligned, range_bytes() of item i, or null: the count pass then
// reads the whole tensor).  The items have been checked.
fh_status classify_with_ranges(const fh_classify_item* items, uint32_t* const* ranges, int32_t count, hipStream_t s);

}  // namespace fh
