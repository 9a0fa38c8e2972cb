// The first half of the channel classification for the elements that a wave holds: pairwise binary64 sums of x and
// x * x over its 1024-element spans, and the range of the values of every 128 elements.  Shared by the pass that does
// nothing else and by the one that quantises the elements as well.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fh_device.hpp"
#include "fh_stages.hpp"

namespace fh {

constexpr int kSpan = 1024;              // elements (or partial sums) per node of the tree's lowest stored level

typedef double f64x2 __attribute__((ext_vector_type(2)));

// ---- lane exchanges of a double ------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// ds_swizzle in bit-mask mode: lane l reads lane (l & 0x1f) ^ XOR inside its half
template <int XOR>
__device__ __forceinline__ double swizzle_f64(double v)
{
    constexpr int pattern = (XOR << 10) | 0x1F;
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_swizzle((int)(uint32_t)u, pattern);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_swizzle((int)(uint32_t)(u >> 32), pattern);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
template <int XOR>
__device__ __forceinline__ double from_lane_xor(double v)
{
    if constexpr (XOR == 1) return dpp_f64<0xB1>(v);        // quad_perm [1,0,3,2]
    else if constexpr (XOR == 2) return dpp_f64<0x4E>(v);   // quad_perm [2,3,0,1]
    else return swizzle_f64<XOR>(v);                          // 4, 8, 16
}
// v[l] + v[l ^ 32]: permlane32_swap of two copies returns {lo half, lo half} and
// {hi half, hi half}; their sum is the same in both halves.
__device__ __forceinline__ double add_across_halves(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    uint32_t a0 = (uint32_t)u, a1 = (uint32_t)(u >> 32), b0 = a0, b1 = a1;
    asm volatile("" : "+v"(b0), "+v"(b1));
    const u32x2 r0 = __builtin_amdgcn_permlane32_swap(a0, b0, false, false);
    const u32x2 r1 = __builtin_amdgcn_permlane32_swap(a1, b1, false, false);
    const uint32_t f0 = r0.x, s0 = r0.y, f1 = r1.x, s1 = r1.y;
    const double first = __builtin_bit_cast(double, ((uint64_t)f1 << 32) | f0);
    const double second = __builtin_bit_cast(double, ((uint64_t)s1 << 32) | s0);
    return first + second;
}

// ---- the span tree ---------------------------------------------------------------------
// In: for each of ROWS rows, the lane's own subtree sums a[r] (of x) and b[r] (of x*x); a row is 64 lanes in element
// order.  Four rows are those of one span, or rows 0 and 1 of one and 2 and 3 of the next (SPANS == 2); two rows are one
// span's.  Out: moment m of span k in lane 2 * k + 4 * m of four rows, in lane 2 * m of two (also elsewhere).
// Exchange levels, in the tree's order:
//   xor 1   keep the rows whose low bit equals the lane's bit 0
//   next    four rows: keep the row whose high bit equals the lane's bit 1
//   next    keep one of the two moments
//   rest    plain butterflies
// followed by the levels that join a span's rows.
template <int SPANS, int ROWS>
__device__ __forceinline__ double span_tree(const double (&a)[ROWS], const double (&b)[ROWS], uint32_t lane)
{
    static_assert((ROWS == 4 && (SPANS == 1 || SPANS == 2)) || (ROWS == 2 && SPANS == 1), "one span or two in four rows, one in two");
    const bool b0 = lane & 1u, b1 = lane & 2u, b2 = lane & 4u;
    // xor 1: rows {b0, b0 + 2} of both moments stay
    double ka[ROWS / 2], kb[ROWS / 2];
#pragma unroll
    for (int j = 0; j < ROWS / 2; ++j) {
        ka[j] = (b0 ? a[2 * j + 1] : a[2 * j]) + from_lane_xor<1>(b0 ? a[2 * j] : a[2 * j + 1]);
        kb[j] = (b0 ? b[2 * j + 1] : b[2 * j]) + from_lane_xor<1>(b0 ? b[2 * j] : b[2 * j + 1]);
    }
    double t;                                                 // one (row, moment) total per lane
    if constexpr (ROWS == 4) {
        // xor 2: row 2 * b1 + b0 stays
        const double ma = (b1 ? ka[1] : ka[0]) + from_lane_xor<2>(b1 ? ka[0] : ka[1]);
        const double mb = (b1 ? kb[1] : kb[0]) + from_lane_xor<2>(b1 ? kb[0] : kb[1]);
        t = (b2 ? mb : ma) + from_lane_xor<4>(b2 ? ma : mb);  // xor 4: moment b2 stays
    } else {
        t = (b1 ? kb[0] : ka[0]) + from_lane_xor<2>(b1 ? ka[0] : kb[0]);      // xor 2: moment b1 stays
        t = t + from_lane_xor<4>(t);
    }
    t = t + from_lane_xor<8>(t);
    t = t + from_lane_xor<16>(t);
    t = add_across_halves(t);
    // rows: (0 + 1) and (2 + 3); of one span in four, their sum too; the row index sits in the lowest lane bits
    t = t + from_lane_xor<1>(t);
    if constexpr (ROWS == 4 && SPANS == 1) t = t + from_lane_xor<2>(t);
    return t;
}
// The sums of one span of four rows as span_tree leaves them, in every lane.
__device__ __forceinline__ void both_moments(double t, uint32_t lane, double& s1, double& s2)
{
    const double other = from_lane_xor<4>(t);                 // lanes with bit 2 clear hold the sum of x, the others that of x*x
    s1 = (lane & 4u) ? other : t;
    s2 = (lane & 4u) ? t : other;
}

// balanced tree over N consecutive values (N a power of two)
template <int N>
__device__ __forceinline__ double local_tree(const double (&v)[N])
{
    double w[N];
#pragma unroll
    for (int i = 0; i < N; ++i) w[i] = v[i];
#pragma unroll
    for (int n = N; n > 1; n /= 2)
#pragma unroll
        for (int i = 0; i < n / 2; ++i) w[i] = w[2 * i] + w[2 * i + 1];
    return w[0];
}

// The counters and the mask of a tensor, by the workgroups of the first pass: THREADS channels each, the first ones.  (All of
// them by one made the pass wait for that one: 26 bf16 tensors of 1 Mi elements with 16384 channels 40.0 us, this way 34.1.)
template <int THREADS>
__device__ __forceinline__ void clear_counters(const Cleared& c, uint32_t block, uint32_t blocks)
{
    const uint32_t parts = ((uint32_t)c.channels + THREADS - 1u) / THREADS, step = (blocks < parts ? blocks : parts) * THREADS;
    if (block >= parts) return;                               // workgroup-uniform
    for (uint32_t i = block * THREADS + threadIdx.x; i < (uint32_t)c.channels; i += step) { c.counts[i] = 0u; c.mask[i] = 0; }
}

// ---- value ranges ------------------------------------------------------------------------
// A piece is what eight neighbouring lanes hold of a span: 128 elements, 128 contiguous bytes in each of the span's
// rows.  Its range is kept as two bf16 numbers, the smallest value rounded down and the largest rounded up, in one
// word: (largest << 16) | smallest.  8 words per span, 0.8 % (bf16: 1.6 %) of what the pass reads.
constexpr int kPieces = 8;                       // of a span
__device__ __forceinline__ uint32_t pack_range(float lowest, float highest)
{
    const uint32_t l = __builtin_bit_cast(uint32_t, lowest), h = __builtin_bit_cast(uint32_t, highest);
    // away from zero: one step up in magnitude unless the low half is empty; towards zero: the low half dropped
    const uint32_t down = (l >> 31) ? (l + 0xffffu) >> 16 : l >> 16, up = (h >> 31) ? h >> 16 : (h + 0xffffu) >> 16;
    return (up << 16) | (down & 0xffffu);
}
// The wave's elements v (row r, 64 lanes with EPL consecutive elements each; what lies past the tensor's end is 0, in
// the range too) are SPANS spans: their sums to partial[0 .. SPANS) and, unless null, their ranges to ranges[], of
// which `here` (or more) exist.  All 64 lanes.
template <int SPANS, int ROWS, int EPL>
__device__ __forceinline__ void leave_moments(const float (&v)[ROWS][EPL], f64x2* partial, uint32_t* ranges, int64_t here,
                                              uint32_t lane)
{
    double a[ROWS], b[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        // the squares are exact, so the fused multiply-add rounds the sum of two of them just as an addition would
        double d[EPL], q[EPL / 2];
#pragma unroll
        for (int j = 0; j < EPL; ++j) d[j] = (double)v[r][j];
#pragma unroll
        for (int j = 0; j < EPL; j += 2) q[j / 2] = __builtin_fma(d[j], d[j], d[j + 1] * d[j + 1]);
        a[r] = local_tree<EPL>(d);
        b[r] = local_tree<EPL / 2>(q);
    }
    const double t = span_tree<SPANS>(a, b, lane);
    const uint32_t k = ROWS == 4 ? (lane >> 1) & 1u : 0u, moment = lane / ROWS;
    if (moment < 2u && (lane & 1u) == 0u && k < (uint32_t)SPANS && (int64_t)k < here)
        reinterpret_cast<double*>(partial + k)[moment] = t;
    if (ranges) {                                             // wave-uniform
#pragma unroll
        for (int s = 0; s < SPANS; ++s) {
            float lowest = __builtin_inff(), highest = -__builtin_inff();
#pragma unroll
            for (int r = s * ROWS / SPANS; r < (s + 1) * ROWS / SPANS; ++r)
#pragma unroll
                for (int j = 0; j < EPL; j += 2) {
                    asm("v_min3_f32 %0, %1, %2, %0" : "+v"(lowest) : "v"(v[r][j]), "v"(v[r][j + 1]));
                    asm("v_max3_f32 %0, %1, %2, %0" : "+v"(highest) : "v"(v[r][j]), "v"(v[r][j + 1]));
                }
            row_minmax<8>(lowest, highest);
            if ((lane & 7u) == 0u && (int64_t)s < here) ranges[s * kPieces + (lane >> 3)] = pack_range(lowest, highest);
        }
    }
}

}  // namespace fh
