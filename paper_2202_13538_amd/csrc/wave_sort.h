// Sort of 64*E 32-bit keys held in the registers of one wavefront (gfx950, wave64), E any number.
//
// Sort position p = lane*E + r (lane-blocked).  A lane first sorts its own E keys, then sorted
// runs of 1, 2, .. 32 lanes are merged two by two: the first step of a merge compares p with its
// mirror image, which leaves two bitonic halves, the following steps halve them across lanes
// (same register, lane ^ mask) until a lane holds a bitonic run of its own, which it sorts in
// registers.  The comparator lists inside a lane are made at compile time: Batcher's merge
// exchange for the first sort, and for bitonic runs the split into even and odd places, both of
// which exist for any length, so the keys need not be padded to a power of two (550 keys take
// E = 10, not 16).
//
// What bounds it is instruction issue (all of these issue once per four cycles and SIMD, except
// ds_swizzle, which shares the LDS pipe, and ds_bpermute, three times as slow as that).  A
// compare-exchange across lanes is one data movement and one v_med3: the median of (mine, yours,
// 0) is the smaller, that of (mine, yours, ~0) the larger key, so the lane's side of the exchange
// is an operand, not a branch or a select.  The last merge, of the two halves of the wave, runs
// on keys that the upper half has sorted in descending order (its keys are inverted before and
// after), so that it needs lane ^ 32 only, which v_permlane32_swap does for two registers at a
// time, and no mirror image across 64 lanes.  For E = 16 that is 1,180 vector instructions and 80
// swizzles, against 1,970 and 96 swizzles + 32 bpermutes with a compare, a mask xor and a select
// per exchange.
#pragma once

#include <utility>

#include "device_util.h"

namespace surel {

// A list of comparators (a < b: the smaller key goes to place a).
template <int N>
struct SortNetwork {
    static constexpr int kMost = N < 2 ? 1 : N * (N - 1) / 2;
    int n = 0;
    int a[kMost] = {};
    int b[kMost] = {};
    constexpr void add(int x, int y) {
        a[n] = x;
        b[n] = y;
        n += 1;
    }
    // Batcher's merge exchange (Knuth, TAOCP 5.2.2 M) on `count` places first, first + stride, ..
    constexpr void add_sort(int first, int stride, int count) {
        if (count < 2) return;
        int top = 1;
        while (top * 2 < count) top *= 2;
        for (int p = top; p > 0; p /= 2) {
            int q = top, r = 0, d = p;
            while (true) {
                for (int i = 0; i + d < count; ++i)
                    if ((i & p) == r) add(first + i * stride, first + (i + d) * stride);
                if (q == p) break;
                d = q - p;
                q /= 2;
                r = p;
            }
        }
    }
    // A bitonic run (rotated in any way) of `count` places: its even and its odd places are bitonic
    // runs.  In the sense of the 0-1 principle its zeros are neighbours on the circle of its places, so
    // where the count is even the two differ by one zero at most; once both are sorted, every even place
    // is compared with the one behind it.  Where it is odd the circle's last place and its first are both
    // even, so the even places have between one zero less and two zeros more than the odd ones; with two
    // more it is the odd places that are compared with the ones behind them, and where one of the two
    // rounds of comparisons has something to do the other has not.  (Odd counts sorted from scratch: 48
    // comparators instead of 34 at 13, 26 instead of 20 at 9, 16 instead of 13 at 7.)
    constexpr void add_bitonic(int first, int stride, int count) {
        if (count < 2) return;
        add_bitonic(first, 2 * stride, (count + 1) / 2);
        add_bitonic(first + stride, 2 * stride, count / 2);
        for (int i = 0; i + 1 < count; i += 2) add(first + i * stride, first + (i + 1) * stride);
        if (count % 2 == 0) return;
        for (int i = 1; i + 1 < count; i += 2) add(first + i * stride, first + (i + 1) * stride);
    }
};
template <int E>
constexpr SortNetwork<E> sort_network() {
    SortNetwork<E> s;
    s.add_sort(0, 1, E);
    return s;
}
template <int E>
constexpr SortNetwork<E> bitonic_network() {
    SortNetwork<E> s;
    s.add_bitonic(0, 1, E);
    return s;
}

template <int A, int B, int E>
__device__ __forceinline__ void compare_places(uint32_t (&x)[E]) {
    const uint32_t lo = min(x[A], x[B]);
    const uint32_t hi = max(x[A], x[B]);
    x[A] = lo;
    x[B] = hi;
}
template <int E, size_t... I>
__device__ __forceinline__ void lane_sort_impl(uint32_t (&x)[E], std::index_sequence<I...>) {
    constexpr SortNetwork<E> net = sort_network<E>();
    (compare_places<net.a[I], net.b[I]>(x), ...);
}
template <int E, size_t... I>
__device__ __forceinline__ void lane_bitonic_impl(uint32_t (&x)[E], std::index_sequence<I...>) {
    constexpr SortNetwork<E> net = bitonic_network<E>();
    (compare_places<net.a[I], net.b[I]>(x), ...);
}
template <int E>
__device__ __forceinline__ void lane_sort(uint32_t (&x)[E]) {
    lane_sort_impl(x, std::make_index_sequence<(size_t)sort_network<E>().n>{});
}
template <int E>
__device__ __forceinline__ void lane_bitonic(uint32_t (&x)[E]) {
    lane_bitonic_impl(x, std::make_index_sequence<(size_t)bitonic_network<E>().n>{});
}

// The smaller of x and y where side is 0, the larger where it is ~0.
__device__ __forceinline__ uint32_t take_side(uint32_t x, uint32_t y, uint32_t side) {
    return max(min(x, y), min(max(x, y), side));  // v_med3_u32
}
// ~0 in the lanes whose bit `bit` is set, 0 in the others.
__device__ __forceinline__ uint32_t lane_side(int lane, int bit) {
    return (lane & bit) != 0 ? ~0u : 0u;
}

// Compare-exchange of every key with that of lane ^ G, ^ G/2, .. ^ 1.
template <int G, int E>
__device__ __forceinline__ void halve_runs(uint32_t (&x)[E], int lane) {
    if constexpr (G >= 1) {
        const uint32_t side = lane_side(lane, G);
#pragma unroll
        for (int r = 0; r < E; ++r) x[r] = take_side(x[r], lane_xor<G>(x[r], lane), side);
        halve_runs<G / 2>(x, lane);
    }
}

// Merges the sorted runs of G/2 lanes to runs of G lanes (G = 2 .. 32).
template <int G, int E>
__device__ __forceinline__ void merge_runs(uint32_t (&x)[E], int lane) {
    const uint32_t side = lane_side(lane, G / 2);
    uint32_t y[E];
#pragma unroll
    for (int r = 0; r < E; ++r) y[r] = lane_xor<G - 1>(x[E - 1 - r], lane);
#pragma unroll
    for (int r = 0; r < E; ++r) x[r] = take_side(x[r], y[r], side);
    halve_runs<G / 4>(x, lane);
    lane_bitonic(x);
}

template <int E>
__device__ __forceinline__ void wave_sort(uint32_t (&x)[E], int lane) {
    const uint32_t invert = lane_side(lane, 32);
#pragma unroll
    for (int r = 0; r < E; ++r) x[r] ^= invert;
    lane_sort(x);
    merge_runs<2>(x, lane);
    merge_runs<4>(x, lane);
    merge_runs<8>(x, lane);
    merge_runs<16>(x, lane);
    merge_runs<32>(x, lane);
#pragma unroll
    for (int r = 0; r < E; ++r) x[r] ^= invert;
    // lanes 0-31 ascend, lanes 32-63 descend: one bitonic run.  permlane32_swap(a, b) exchanges
    // the upper half of a with the lower half of b.
#pragma unroll
    for (int r = 0; r + 1 < E; r += 2) {
        const auto t = __builtin_amdgcn_permlane32_swap(x[r], x[r + 1], false, false);
        const auto u = __builtin_amdgcn_permlane32_swap(min(t[0], t[1]), max(t[0], t[1]), false, false);
        x[r] = u[0];
        x[r + 1] = u[1];
    }
    if constexpr (E % 2 == 1) {
        const auto t = __builtin_amdgcn_permlane32_swap(x[E - 1], x[E - 1], false, false);
        x[E - 1] = take_side(t[0], t[1], invert);
    }
    halve_runs<16>(x, lane);
    lane_bitonic(x);
}

}  // namespace surel
