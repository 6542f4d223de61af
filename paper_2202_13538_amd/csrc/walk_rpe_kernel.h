// Walk sampling and RPE in one kernel (Sec. 3.2: the RPE is computed on the fly as the walks
// get sampled; Algorithm 1, walk and RPE steps).
//
// A wavefront handles one seed at a time: it walks the M walkers (128 at a time, two per
// lane) into an LDS copy of the seed's walk block, streams the block out, turns the same LDS
// words into sort keys, sorts them in registers and derives the seed's rows (walk_rpe_core.h,
// rpe_rows.h).  The walk waits on memory almost all the time and the sort is pure
// VALU work, so the two overlap across the waves of a compute unit, and the walks are never
// read back from HBM.
//
// Where a seed's rows go is a prefix sum over all earlier seeds.  The kernel is persistent and
// uses the worker / scanner scheme of lookback.h: workers take seeds in increasing order, a
// worker publishes a seed's row count as soon as the sort has it, keeps the sorted keys in
// registers, and only writes the rows out after it has walked and sorted its NEXT seed: by then
// the scanner wave has long published the offset, so nobody waits in practice.  Why every wait
// ends, and how waits are bounded, is argued in lookback.h.
#pragma once

#include "device_util.h"
#include "kernels.h"
#include "lookback.h"
#include "prune_set.h"
#include "walk_rpe_core.h"

namespace surel {

// E = sort keys per lane (64*E >= fused_keys(M, m)).  The waves of a workgroup share the LDS
// allocation and the chunk word (with kCodes also a cache of the hash set), nothing else.
// kCodes: every finished row's count vector is looked up in the hash set while the row still
// lies in LDS (Algorithm 1's last step, pruning, done on the fly as well), and its number there
// goes to code; cnt may then be null.
// Registers: with fewer than 16 waves on a compute unit the gathers wait longer, so E > 8 with kCodes
// spills: 6 of 126 vector registers at E = 9 and 10, 14 of 128 at 12, 17 at 13, 22 at 14, 32 at 16 (the plain
// forms none, 2 in one of E = 16).  Scalar ones go to lanes of a vector register, 48 to 69 in the plain forms and
// 166 to 189 with kCodes, whose look-up is there for five lengths of vector.
template <int E, int kRec, bool kCodes>
__global__ __launch_bounds__(E <= 16 ? 1024 : 512) void walk_rpe_kernel(FusedJob f,
                                                                        uint64_t* __restrict__ lb,
                                                                        int32_t* __restrict__ code,
                                                                        VectorSet set) {
    extern __shared__ __align__(16) uint32_t lds32[];
    __shared__ unsigned long long chunk;
    __shared__ bool scans;
    __shared__ __align__(16) uint32_t set_cache[kCodes ? kDirectWords + FusedTables::kHashed : 1];

    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n_waves = (int)(blockDim.x >> 6);
    // One draw per workgroup gives it its first run of items, and the role of the scanner to the
    // first wave of the workgroup that draws item 0.  (A draw of its role by every wave, 4,096
    // additions to one address, took 50 us before any seed was walked.)
    if (threadIdx.x == 0) {
        const uint64_t first = atomicAdd(reinterpret_cast<unsigned long long*>(lb),
                                         (unsigned long long)n_waves);
        scans = first == 0;
        chunk = (first + n_waves) << 32 | first;
    }
    if constexpr (kCodes) set_cache_clear(set_cache, kDirectWords + FusedTables::kHashed, (int)threadIdx.x, (int)blockDim.x);
    __syncthreads();                     // the only workgroup-wide barrier of the kernel
    const LookbackScratch scr = lookback_scratch(f.n_seeds);
    int64_t* base = lookback_base(lb);
    uint16_t* status = lookback_status(lb, scr);
    if (scans && wave == 0) {
        scan_counts(status, scr.n_groups, base, f.rpe_off + f.n_seeds, f.h_total, f.spin_limit, f.err,
                    lane);
        return;
    }

    const int L = f.m + 1;
    // the seed's walks [M][L] while it is walked, the rows of the seed before while they go out
    uint32_t* wave_lds = lds32 + wave * f.lds_words_per_wave;

    // the seed whose offset and rows are not written yet: its sorted keys stay in registers
    uint32_t x[E];
    RpeRowScan sc{};
    int64_t held = -1;
    for (;;) {
        const int64_t i = take_item<kGroup>(&chunk, lb, lane);
        const bool more = i < f.n_seeds;
        uint32_t y[E];
        RpeRowScan sc_y{};  // no rows
        if (more) {
            const int32_t u = __builtin_amdgcn_readfirstlane(f.seeds[i]);
            if (u < 0 || u >= f.g.n_nodes) {
                fused_bad_seed(f, i, lane);
#pragma unroll
                for (int r = 0; r < E; ++r) y[r] = pad_key(lane);
            } else {
                fused_walk_and_sort<E, kRec>(f, i, u, reinterpret_cast<int32_t*>(wave_lds), lane, y);
                sc_y = rpe_scan_rows<E>(y, lane);
            }
            // the count goes out before anything is waited for: publishing never depends on others
            if (lane == 0) store_u16_agent(status + i, (uint32_t)sc_y.n_rows + 1u);
        }
        // the seed before this one: its offset has had a whole walk and a sort to arrive
        if (held >= 0) {
            const int64_t off = wait_offset(status, base, held, f.spin_limit, lane);
            if (off < 0) {
                if (lane == 0) {
                    atomicOr(f.err, kDevStall);
                    int64_t* h_total = lookback_host(lb);
                    if (h_total) h_total[1] = 1;
                }
                return;
            }
            if (lane == 0) f.rpe_off[held] = off;
            if (f.ids != nullptr && sc.n_rows > 0) {
                if (off + sc.n_rows > f.cap_rows) {
                    if (lane == 0) atomicOr(f.err, kDevCapacity);
                } else {
                    rpe_write_rows<E>(
                        x, sc, lane, L, (uint32_t)f.M, wave_lds, f.lds_rows, off, f.ids, f.cnt, f.past,
                        [&](int row0, int n, const uint16_t* cnt16, uint32_t* free_words) {
                            // every row's number in the set of distinct vectors
                            if constexpr (kCodes)
                                rows_numbers_any<FusedTables>(n, lane, L, cnt16,
                                                 reinterpret_cast<uint16_t*>(free_words), set_cache, set,
                                                 code + off + row0);
                        });
                }
            }
        }
        if (!more) break;
        copy_keys(x, y);
        sc = sc_y;
        held = i;
    }
}

template <int E, int kRec, bool kCodes>
hipError_t launch_walk_rpe_erc(hipStream_t stream, int max_lds_bytes, int n_cu, FusedJob f,
                                      uint64_t* lb, int32_t* code, const VectorSet& set) {
    const void* fn = reinterpret_cast<const void*>(walk_rpe_kernel<E, kRec, kCodes>);
    // A workgroup has as many waves as LDS (160 KB) and registers allow a compute unit, 16 at
    // most, so that a compute unit holds one such workgroup (two, where 32 waves fit).
    // (Kernels with few registers could have 20 or 24 waves in two or more smaller workgroups,
    // and were measured with them on the 2.9M-node graph: M = 50, m = 4, where 20 waves fit,
    // takes 8.2 ms as one workgroup of 16, 9.1 as two of 8, 11.9 as five of 4, and 11.3 as two
    // of 10, of which the second never starts beside the first: a workgroup's waves go to the
    // four SIMDs in turn, and two of 10 ask two of the SIMDs for six waves when five fit.
    // M = 25: 6.7 ms as 16, 6.9 as two of 12.  Only at M = 12 are two of 12 ahead, 5.4 against
    // 5.6 ms.  Registers held to 64, for two workgroups of 16, spill 27 of them where E = 10: 100,000
    // nodes, M = 61, m = 9 take 0.88 ms, 0.67 as one of 16.)
    hipFuncAttributes attr;
    hipError_t rc = hipFuncGetAttributes(&attr, fn);
    if (rc != hipSuccess) return rc;
    const int regs = attr.numRegs > 0 ? attr.numRegs : 128;
    constexpr int kMaxW = E <= 16 ? 16 : 8;
    int W = 4 * (512 / ((regs + 7) / 8 * 8));
    if (W > kMaxW) W = kMaxW;
    // every wave has its share of what the static part leaves of the LDS
    const int lds_words = (160 * 1024 - (int)attr.sharedSizeBytes) / 4;
    fused_lds_plan(&f, lds_words / W & ~3);
    if (W > lds_words / f.lds_words_per_wave) W = lds_words / f.lds_words_per_wave;
    if (W < 1 || f.lds_rows < 1) return hipErrorInvalidValue;
    const size_t lds_bytes = (size_t)W * f.lds_words_per_wave * 4;
    if (lds_bytes + attr.sharedSizeBytes > (size_t)max_lds_bytes) return hipErrorInvalidValue;
    if (lds_bytes > 48 * 1024) {
        rc = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (rc != hipSuccess) return rc;
    }
    // as many workgroups as the device holds at once, or fewer if the job is small: one wave
    // for the scanner and at most one per seed
    int per_cu = 0;
    rc = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, W * kWave, lds_bytes);
    if (rc != hipSuccess) return rc;
    if (per_cu < 1) return hipErrorInvalidValue;
    int64_t blocks = (f.n_seeds + 1 + W - 1) / W;
    if (blocks > (int64_t)per_cu * n_cu) blocks = (int64_t)per_cu * n_cu;
    if (blocks * W < 2) blocks = 2;  // the scanner and at least one worker

    rc = launch_lookback_clear(stream, lb, f.n_seeds, f.rpe_off + f.n_seeds, f.h_total);
    if (rc != hipSuccess) return rc;
    hipLaunchKernelGGL((walk_rpe_kernel<E, kRec, kCodes>), dim3((unsigned)blocks), dim3(W * kWave),
                       lds_bytes, stream, f, lb, code, set);
    return hipGetLastError();
}

// kCodes: true in walk_rpe_ids.hip, false in walk_rpe.hip (two files, which compile at the same time).
template <bool kCodes, int E>
hipError_t launch_walk_rpe_e(hipStream_t stream, int max_lds_bytes, int n_cu, const FusedJob& f,
                             int rec_format, uint64_t* lb, int32_t* code, const VectorSet& set) {
#define SUREL_WR_CASE(REC_) \
    return launch_walk_rpe_erc<E, REC_, kCodes>(stream, max_lds_bytes, n_cu, f, lb, code, set)
    if (f.g.rec == nullptr) SUREL_WR_CASE(kRecNone);
    if (rec_format == kRecPacked) SUREL_WR_CASE(kRecPacked);
    if (rec_format == kRecShort) SUREL_WR_CASE(kRecShort);
    SUREL_WR_CASE(kRecWide);
#undef SUREL_WR_CASE
}

template <bool kCodes>
hipError_t launch_walk_rpe_form(hipStream_t stream, int max_lds_bytes, int n_cu, const FusedJob& f,
                                int rec_format, uint64_t* lb, int32_t* code, const VectorSet& set) {
    const int n_key = fused_keys(f.M, f.m);
#define SUREL_WR_SIZE(E_) \
    if (n_key <= kWave * (E_)) return launch_walk_rpe_e<kCodes, E_>(stream, max_lds_bytes, n_cu, f, rec_format, lb, code, set);
    SUREL_FOR_SORT_SIZES(SUREL_WR_SIZE)
#undef SUREL_WR_SIZE
    return hipErrorInvalidValue;
}

// walk_rpe_ids.hip: the form with look-ups
hipError_t launch_walk_rpe_codes(hipStream_t stream, int max_lds_bytes, int n_cu, const FusedJob& f,
                                 int rec_format, uint64_t* lb, int32_t* code, const VectorSet& set);

}  // namespace surel
