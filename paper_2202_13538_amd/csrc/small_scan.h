// Offsets of variable-size blocks inside ONE launch for small jobs: every workgroup publishes its
// number of rows and adds up the numbers of the workgroups before it, most of which run at the same
// time.  (Large jobs use a scanner wave, lookback.h, or a counting launch and a scan of its counts:
// there a workgroup cannot look at everybody before it.)
//
// A word per workgroup holds (tag << 32 | rows).  The tag is the number of the launch, kept on
// the device and moved on by the launch itself, so nothing has to be cleared before the next
// launch, and a launch that was captured into a graph finds a new number at every replay.  The
// number is moved on by the workgroup that is the last to say "done"; a workgroup says so once it
// has read the number and waits for nobody any more, so no word of an earlier launch is ever
// taken for one of this launch.
// No workgroup depends on another one.  Which workgroups the device holds at a time is not in this
// code's hands: launches of other contexts may fill a die while the workgroups of this launch that
// the others wait for are still to start there, and those launches may be waiting in the same way.
// So whoever has polled kHelpAfter times (or as often as the spin limit allows) for a number works
// it out itself, publishes it in its owner's place (the owner, once it runs, publishes the same
// number) and looks again.  There are at most as many numbers to work out as workgroups before it,
// so every workgroup comes to its end, with all of its rows.  Working a number out is written for
// few instructions and registers, not for speed: it stands in kernels that hardly ever run it.
// (The workgroup's own work done over for another one, in a loop around it, made everybody pay:
// what the compiler moved out of that loop took the walks from 47 to 93 registers, and 32 pairs
// 23.7 us instead of 23.0.)
#pragma once

#include "device_util.h"

namespace surel {

constexpr int kSmallScanMax = 4096;  // workgroups of a launch, at most
constexpr int kDoneParts = 32;
// Polls before a workgroup helps: milliseconds, a hundred times what a launch of this kind takes.
constexpr uint32_t kHelpAfter = 4096;

struct SmallScan {
    uint32_t launch;                  // number of the next launch
    uint32_t unused[31];
    // Workgroups of the present launch that wait no more: at the first level workgroup i counts
    // in word i % kDoneParts, each in a cache line of its own, and whoever fills a word counts in
    // the last one.  (A thousand additions to ONE word take 13 us, one after the other.)
    uint32_t done[(kDoneParts + 1) * 32];
    uint64_t rows[kSmallScanMax];     // tag << 32 | rows of the workgroup
};

__device__ __forceinline__ uint32_t small_scan_tag(const SmallScan* s) {
    // + 1: the words of a new context are zero, which is no tag
    return __hip_atomic_load(&s->launch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u;
}

// One lane publishes the rows of workgroup `at`.
__device__ __forceinline__ void small_scan_publish(SmallScan* s, int at, uint32_t tag, uint32_t rows) {
    __hip_atomic_store(&s->rows[at], ((uint64_t)tag << 32) | rows, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

// Rows of the workgroups before `at` (one wavefront calls it).  rows_of(j): works the rows of
// workgroup j out (the wavefront's lanes together, the same result in each).
template <typename RowsOf>
__device__ __forceinline__ int64_t small_scan_before(SmallScan* s, int at, uint32_t tag,
                                                     uint32_t spin_limit, int lane,
                                                     RowsOf&& rows_of) {
    constexpr int kWords = 8;  // words a lane has in flight
    uint32_t polls = min(spin_limit, kHelpAfter);
    uint64_t sum = 0;
    for (int t0 = 0; t0 < at; t0 += kWords * kWave) {
        for (uint32_t spin = 0;; ++spin) {
            int missing = -1;
            uint64_t part = 0;
            uint64_t w[kWords];
#pragma unroll
            for (int u = 0; u < kWords; ++u) {
                const int t = t0 + u * kWave + lane;
                w[u] = (uint64_t)tag << 32;
                if (t < at)
                    w[u] = __hip_atomic_load(&s->rows[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
#pragma unroll
            for (int u = 0; u < kWords; ++u) {
                missing = (uint32_t)(w[u] >> 32) != tag ? t0 + u * kWave + lane : missing;
                part += (uint32_t)w[u];
            }
            const uint64_t lanes = __ballot(missing >= 0);
            if (lanes == 0ull) {
                sum += part;
                break;
            }
            if (spin >= polls) {
                // of several that are missing, one that depends on `at`: helpers share them out
                const int turn = at & (kWave - 1);
                const uint64_t turned = (lanes >> turn) | (lanes << ((kWave - turn) & (kWave - 1)));
                const int from = (__builtin_ctzll(turned) + turn) & (kWave - 1);
                const int j = (int)wave_bcast_u32((uint32_t)missing, from);
                const uint32_t rows = rows_of(j);
                if (lane == 0) small_scan_publish(s, j, tag, rows);
                polls = 0;
            }
            __builtin_amdgcn_s_sleep(1);
        }
    }
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)sum, d, kWave);
        const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(sum >> 32), d, kWave);
        sum += ((uint64_t)hi << 32) | lo;
    }
    return (int64_t)sum;
}

// One lane of workgroup `at` calls it when the workgroup waits no more.
__device__ __forceinline__ void small_scan_done(SmallScan* s, int at, uint32_t tag, int n_groups) {
    const int part = at % kDoneParts;
    const uint32_t n_part = (uint32_t)((n_groups - part + kDoneParts - 1) / kDoneParts);
    const uint32_t n_parts = (uint32_t)min(n_groups, kDoneParts);
    uint32_t* mine = &s->done[part * 32];
    uint32_t* last = &s->done[kDoneParts * 32];
    if (atomicAdd(mine, 1u) + 1u != n_part) return;
    __hip_atomic_store(mine, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (atomicAdd(last, 1u) + 1u != n_parts) return;
    __hip_atomic_store(last, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&s->launch, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace surel
