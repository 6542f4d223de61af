// Device-side helpers shared by the HIP kernels of libsurel (gfx950, wave64 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace surel {

constexpr int kWave = 64;

// Bits of the sticky device error word (same values as SUREL_DEV_* in the public header).
constexpr uint32_t kDevBadSeed = 0x01u;
constexpr uint32_t kDevBadGraph = 0x02u;
constexpr uint32_t kDevBadWalk = 0x04u;
constexpr uint32_t kDevBadQuery = 0x08u;
constexpr uint32_t kDevSetTooLarge = 0x10u;
constexpr uint32_t kDevCapacity = 0x20u;
constexpr uint32_t kDevBadTable = 0x40u;
constexpr uint32_t kDevBadSizes = 0x80u;
constexpr uint32_t kDevStall = 0x100u;

__device__ __forceinline__ int lane_id() {
    return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

// Orders LDS traffic between the lanes of ONE wavefront.  LDS instructions of a wave execute
// in issue order, so no hardware barrier is needed; the fence keeps the compiler from moving
// LDS accesses across this point.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Waits until every load and store that this wavefront has issued to memory is done, and keeps the
// compiler from moving memory accesses across this point: what is read behind it was not read before it,
// and whoever sees a store behind it sees the (write-through) stores before it.
__device__ __forceinline__ void wait_memory() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// A register with some value, for a variable that is set on a part of the ways to where it is used and does
// not matter on the others (an unset one would make that use undefined; to set it takes an instruction).
__device__ __forceinline__ uint32_t any_value() {
    uint32_t x;
    asm volatile("" : "=v"(x));
    return x;
}

// Raise bits of the error word: one atomic per wave at most, none in the common case.
__device__ __forceinline__ void raise_error(uint32_t* err, bool cond, uint32_t bit) {
    if (__ballot(cond) != 0ull) {
        if (lane_id() == 0) atomicOr(err, bit);
    }
}

// Moves a value between lanes by DPP (part of the vector unit, folded into the consuming
// instruction where that allows it); lanes without a source get `old`.
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ uint32_t dpp_move(uint32_t old, uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)x, CTRL, ROWS, 0xF, false);
}
// The same for patterns in which every lane has a source.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_permute(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);
}

// Value of `x` held by lane (lane ^ MASK), MASK a compile-time constant in 1..31: DPP where the
// pattern allows it, the LDS crossbar's swizzle (no LDS memory is touched) otherwise.
template <int MASK>
__device__ __forceinline__ uint32_t lane_xor(uint32_t x, int lane) {
    static_assert(MASK >= 1 && MASK < 32, "mask out of range");
    if constexpr (MASK == 1) {
        return dpp_permute<0xB1>(x);   // quad_perm [1,0,3,2]
    } else if constexpr (MASK == 2) {
        return dpp_permute<0x4E>(x);   // quad_perm [2,3,0,1]
    } else if constexpr (MASK == 3) {
        return dpp_permute<0x1B>(x);   // quad_perm [3,2,1,0]
    } else if constexpr (MASK == 7) {
        return dpp_permute<0x141>(x);  // row_half_mirror
    } else if constexpr (MASK == 8) {
        return dpp_permute<0x128>(x);  // row_ror:8
    } else if constexpr (MASK == 15) {
        return dpp_permute<0x140>(x);  // row_mirror
    } else {
        // swizzle, bit mode: new lane = ((lane & and) | or) ^ xor inside each group of 32
        return (uint32_t)__builtin_amdgcn_ds_swizzle((int)x, (MASK << 10) | 0x1F);
    }
}

// The value of lane `src_lane` (the same in every lane).
__device__ __forceinline__ uint32_t wave_bcast_u32(uint32_t v, int src_lane) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, src_lane);
}

// The value of the lane below (lane 0: its own).
__device__ __forceinline__ uint32_t wave_from_lane_below(uint32_t v) {
    return dpp_move<0x138>(v, v);  // wave_shr:1
}

// Inclusive prefix sum over the 64 lanes: inside rows of 16 lanes by shifts of 1, 2, 4 and 8, then
// the last lane of a row to the row behind it, then lane 31 to the upper half.
__device__ __forceinline__ uint32_t wave_incl_sum(uint32_t v) {
    v += dpp_move<0x111>(0u, v);       // row_shr:1
    v += dpp_move<0x112>(0u, v);
    v += dpp_move<0x114>(0u, v);
    v += dpp_move<0x118>(0u, v);
    v += dpp_move<0x142, 0xA>(0u, v);  // row_bcast:15 to rows 1 and 3
    v += dpp_move<0x143, 0xC>(0u, v);  // row_bcast:31 to rows 2 and 3
    return v;
}

// Copies n 32-bit words from global memory to LDS with `threads` threads, numbered tid.  Loads
// are issued U at a time before any of them is waited for, so a copy costs
// ceil(n / (threads*U)) memory round trips instead of one per `threads` words.
template <int U>
__device__ __forceinline__ void stage_words(uint32_t* dst, const uint32_t* __restrict__ src, int n,
                                            int tid, int threads = kWave) {
    for (int t0 = 0; t0 < n; t0 += threads * U) {
        uint32_t v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int t = t0 + u * threads + tid;
            v[u] = t < n ? src[t] : 0u;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int t = t0 + u * threads + tid;
            if (t < n) dst[t] = v[u];
        }
    }
}

// Philox-4x32 with 10 rounds (Salmon et al., SC'11): counter c[0..3], key (k0, k1).
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1, uint32_t out[4]) {
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0;  // one v_mad_u64_u32 each
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c1 ^ k0;
        const uint32_t n2 = (uint32_t)(p0 >> 32) ^ c3 ^ k1;
        c0 = n0;
        c1 = (uint32_t)p1;
        c2 = n2;
        c3 = (uint32_t)p0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    out[0] = c0;
    out[1] = c1;
    out[2] = c2;
    out[3] = c3;
}

// r mod d for d >= 1, exact, in about 13 instructions: the quotient from a reciprocal of d with
// more than 40 good bits (a single-precision reciprocal and one Newton step in double precision)
// is below 2^32 and lowered by 2^-10, far more than its error, so it is the true one or one less,
// which the last step mends.
__device__ __forceinline__ uint32_t mod_u32(uint32_t r, uint32_t d) {
    const double dd = (double)d;
    double y = (double)__builtin_amdgcn_rcpf((float)d);
    y = __builtin_fma(__builtin_fma(-dd, y, 1.0), y, y);
    const uint32_t q = (uint32_t)__builtin_fma((double)r, y, -0x1p-10);
    const uint32_t rest = r - q * d;
    return min(rest, rest - d);
}

// floor(x / d) for 0 <= x < 4096 and 1 <= d <= 16 with magic = 65536 / d + 1.
// Exact because x * (magic * d - 65536) <= x * d < 65536.
__device__ __forceinline__ uint32_t small_div(uint32_t x, uint32_t magic) {
    return (x * magic) >> 16;
}

// floor(x / d) for x * d < 2^32 with magic = 2^32 / d + 1 (d >= 2; the host passes it in).
__device__ __forceinline__ uint32_t div_magic32(uint32_t x, uint32_t magic) {
    return __umulhi(x, magic);
}

}  // namespace surel
