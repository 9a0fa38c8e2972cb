// Several tensors per launch: descriptors travel by value in the kernel-argument segment and a
// workgroup finds its tensor by a scalar search over the exclusive prefix sums of the tensors'
// workgroup counts (entries past the last tensor repeat the total).
#pragma once

#include <hip/hip_runtime.h>
#include <limits.h>
#include <stdint.h>

#include <type_traits>

namespace fh {

// Tensors per launch: as many as the largest descriptor (the routed quantiser's, 152 bytes) lets into 4 KiB of kernel
// arguments (fh_kernels.hpp holds it to that).  A stage's serial kernels (the Huffman tables and codes) take as long
// for a full launch as for one tensor: the whole chain on 24 activations takes 871 us in one launch per stage, 1047 in
// launches of 16.
constexpr int kBatch = 26;
constexpr int kBatchStated = 16;                   // what the *_batch_capacity() calls promise

template <typename Item> struct Batch {
    int32_t  count;
    uint32_t block_start[kBatch + 1];
    Item     item[kBatch];
};

// index of the tensor workgroup `bid` works on; `local` = its workgroup number inside that tensor
template <typename Item>
__device__ __forceinline__ int batch_item(const Batch<Item>& b, uint32_t bid, uint32_t& local)
{
    int lo = 0, hi = b.count;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (b.block_start[mid] <= bid) lo = mid; else hi = mid;
    }
    local = bid - b.block_start[lo];
    return lo;
}

// host side: append an item that needs `blocks` workgroups; false when the launch is full
template <typename Item>
inline bool push(Batch<Item>& b, const Item& item, int64_t blocks)
{
    static_assert(sizeof(Batch<Item>) <= 4096, "kernel arguments must fit the 4 KiB segment");
    if (b.count == kBatch || (uint64_t)b.block_start[b.count] + (uint64_t)blocks > (uint64_t)INT_MAX) return false;
    b.item[b.count] = item;
    b.block_start[b.count + 1] = b.block_start[b.count] + (uint32_t)blocks;
    ++b.count;
    return true;
}
template <typename Item> inline void seal(Batch<Item>& b)
{
    for (int k = b.count + 1; k <= kBatch; ++k) b.block_start[k] = b.block_start[b.count];
}
template <typename Item> inline void reset(Batch<Item>& b) { b.count = 0; b.block_start[0] = 0; }

// A launch of one tensor carries its descriptor alone.  Up to 112 bytes of arguments a launch is enqueued in 2.8 us, with 120 in 3.7,
// with 1000 to 4000 in 4.1 to 4.3 (launches of an empty kernel in a row); hidden arguments, the grid's size for one, count.  What
// that is worth where calls follow one another, with the batch's arguments and with these, us: one fp32 tensor of 1 MiB quantised and restored
// 9.4 and 6.6, of 16 MiB 12.2 and 9.7, of 64 MiB 28.9 and 28.4; routed, 0.8 MB, 10.6 and 7.0, 3.2 MB 10.9 and 7.7; classified, 1 MB 10.6 and
// 6.4, 19 MB 19.2 and 15.2, 77 MB 27.2 and 24.4 (the first pass 0.4 of it, the level between 0.3, the count pass 0.5, of wide tensors the masks 1.5);
// Huffman-coded, 1 Mi symbols, 32.1 and 31.1 (histogram 0.6, codes 0.2, count and write 0.9), 32 Mi 65.6 and 65.0; decoded 26.7 and
// 26.4, 35.0 and 34.7; the whole chain, 0.3 MB 95.6 and 81.6, 77 MB 146 and 141 (preparing 1.1, quantiser with first pass 0.7).  Under a caller
// that takes longer to make its calls than a launch to be enqueued it is worth nothing.  Left out where nothing is gained: launches with tiles in runs
// (40 us and more), with limits apart, the Huffman scan and the write pass behind it (315 M symbols 329 and 329), decoding in whole lines; the sparse
// stage's descriptor is longer; the routed quantiser's is shortened (fh_kernels.hpp).
constexpr size_t kOneLaunchArgs = 112;
template <typename Item> struct One {
    Item item;
};
// the descriptor of workgroup `bid`, and the workgroup's number inside that tensor
template <typename Item>
__device__ __forceinline__ const Item& item_of(const Batch<Item>& b, uint32_t bid, uint32_t& local) { return b.item[batch_item(b, bid, local)]; }
template <typename Item>
__device__ __forceinline__ const Item& item_of(const One<Item>& b, uint32_t bid, uint32_t& local) { local = bid; return b.item; }
// the same where every tensor has one workgroup
template <typename Item> __device__ __forceinline__ const Item& item_of(const Batch<Item>& b, uint32_t bid) { return b.item[bid]; }
template <typename Item> __device__ __forceinline__ const Item& item_of(const One<Item>& b, uint32_t) { return b.item; }
// host side: `launch` with the arguments that the launch needs
template <typename Item, typename Launch> inline void with_arguments(const Batch<Item>& b, const Launch& launch)
{
    static_assert(sizeof(One<Item>) <= kOneLaunchArgs, "the descriptor of one tensor is a short argument segment");
    if (b.count == 1) launch(One<Item>{b.item[0]});
    else launch(b);
}
#define FH_ARGS std::decay_t<decltype(args)>

}  // namespace fh
