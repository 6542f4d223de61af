// Walks and RPE of few seeds (Sec. 3.2) in one launch, a wavefront per seed, as many seeds as the
// device has room for at a time.
//
// The kernel for many seeds (walk_rpe_kernel.h) has waves that draw seeds, a scanner wave, and scratch
// that a launch of its own clears; on large graphs it reads neighbour records that another launch
// makes.  With a seed or less per wave of the chip none of that pays: the time is the chain of one
// seed (its walks' dependent gathers, the sort, the offset, the rows) plus every launch around it.
// Here a workgroup adds up the row counts of its seeds, publishes the sum and adds up those of the
// workgroups before it (small_scan.h), and the walks read the CSR as it is.
// Measured, passes with the join behind it: 4,096 seeds of M = 50, m = 4 56 us, 76 with the kernel
// for many seeds; 2,000 seeds of M = 100 on a 2.9M-node graph 70 us instead of 89.
// What bounds it: line fetches, two a step (row_ptr, col_idx), with half as many walks in flight as a full
// device has.  These 2,000 seeds take 27 us with m = 4: 9 with m = 1, then 3, 7 and 8 for steps two to four;
// 18 with M = 50, 47 with M = 200, 8 with one walk.  0.83 M lines are read, 44 G/s over the last 19 us,
// where a device full of gathers reads 56 from an array of this size.  New seeds take 1 us longer.
#include "device_util.h"
#include "kernels.h"
#include "small_scan.h"
#include "walk_rpe_core.h"

namespace surel {

constexpr int small_walk_waves(int E) { return E <= 16 ? 16 : 8; }  // of a compute unit, by registers

// Rows of seed number i, for a workgroup that helps another one: its walks once more, and every
// entry compared with those before it.  block: LDS of the wave, fused_block_words(M, m) words.
__device__ __forceinline__ uint32_t small_walk_rows(const FusedJob& f, int64_t i, int32_t* block,
                                                    int lane) {
    const int32_t u = __builtin_amdgcn_readfirstlane(f.seeds[i]);
    if (u < 0 || u >= f.g.n_nodes) return 0;
    const int L = f.m + 1, n = f.M * L;
    int32_t u_lo, u_deg;
    seed_row(f.g, u, &u_lo, &u_deg);
#pragma unroll 1
    for (int w0 = 0; w0 < f.M; w0 += kWave) {
        const int w[1] = {w0 + lane};
        const bool active[1] = {w[0] < f.M};
        int32_t* const row[1] = {block + (active[0] ? w[0] : f.M) * L};
        walk_many<kRecNone, 1, false>(f.g, u, u_lo, u_deg, w, active, f.m, f.key0, f.key1, row,
                                      [](int, int32_t) {});
    }
    wave_sync();
    uint32_t rows = 0;
#pragma unroll 1
    for (int t0 = 0; t0 < n; t0 += kWave) {
        const int t = t0 + lane;
        const int32_t v = block[min(t, n - 1)];
        bool first = t < n;
#pragma unroll 1
        for (int s = 0; s < min(t0 + kWave, n); ++s) first = first && !(s < t && block[s] == v);
        rows += (uint32_t)__popcll(__ballot(first));
    }
    wave_sync();
    return rows;
}

template <int E>
__global__ __launch_bounds__(small_walk_waves(E) * kWave) void walk_rpe_small_kernel(
    FusedJob f, SmallScan* __restrict__ ss) {
    extern __shared__ __align__(16) uint32_t lds32[];
    __shared__ int32_t rows_of[16];
    __shared__ int64_t s_base;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n_waves = (int)(blockDim.x >> 6);
    const int64_t i = (int64_t)blockIdx.x * n_waves + wave;
    uint32_t tag = 0;
    if (wave == 0) tag = small_scan_tag(ss);
    const int L = f.m + 1;
    uint32_t* wave_lds = lds32 + wave * f.lds_words_per_wave;
    uint32_t x[E];
    RpeRowScan sc{};  // no rows
    if (i < f.n_seeds) {
        const int32_t u = __builtin_amdgcn_readfirstlane(f.seeds[i]);
        if (u < 0 || u >= f.g.n_nodes) {
            fused_bad_seed(f, i, lane);
        } else {
            fused_walk_and_sort<E, kRecNone>(f, i, u, reinterpret_cast<int32_t*>(wave_lds), lane, x);
            sc = rpe_scan_rows<E>(x, lane);
        }
    }
    if (lane == 0) rows_of[wave] = sc.n_rows;
    __syncthreads();
    if (wave == 0) {
        const uint32_t mine = lane < n_waves ? (uint32_t)rows_of[lane] : 0u;
        const uint32_t sum = wave_bcast_u32(wave_incl_sum(mine), kWave - 1);
        const int at = (int)blockIdx.x;
        if (lane == 0) small_scan_publish(ss, at, tag, sum);
        const int64_t before = small_scan_before(ss, at, tag, f.spin_limit, lane, [&](int j) {
            uint32_t rows = 0;  // (the wave's LDS is free: its keys are in registers)
            const int64_t last = min((int64_t)(j + 1) * n_waves, f.n_seeds);
            for (int64_t s = (int64_t)j * n_waves; s < last; ++s)
                rows += small_walk_rows(f, s, reinterpret_cast<int32_t*>(wave_lds), lane);
            return rows;
        });
        if (lane == 0) {
            small_scan_done(ss, at, tag, (int)gridDim.x);
            s_base = before;
            if (at == (int)gridDim.x - 1) {
                f.rpe_off[f.n_seeds] = before + sum;
                if (f.h_total) *f.h_total = before + sum;
            }
        }
    }
    __syncthreads();
    if (i >= f.n_seeds) return;
    int64_t off = s_base;
    for (int w = 0; w < wave; ++w) off += rows_of[w];
    if (lane == 0) f.rpe_off[i] = off;
    if (f.ids == nullptr || sc.n_rows == 0) return;
    if (off + sc.n_rows > f.cap_rows) {
        if (lane == 0) atomicOr(f.err, kDevCapacity);
        return;
    }
    rpe_write_rows<E>(x, sc, lane, L, (uint32_t)f.M, wave_lds, f.lds_rows, off, f.ids, f.cnt, false,
                      [](int, int, const uint16_t*, uint32_t*) {});
}

// Waves of a workgroup: the seeds spread over all compute units, one workgroup on each.
static int small_walk_group(int n_cu, int64_t n_seeds) {
    int w = 1;
    while ((int64_t)n_cu * w < n_seeds) w *= 2;
    return w;
}

bool walk_rpe_is_small(int n_cu, int64_t n_seeds, int32_t M, int32_t m) {
    const int n_key = fused_keys(M, m);
    if (n_key > 64 * 32) return false;
    const int most = small_walk_waves(n_key <= 64 * 16 ? 16 : 32);
    return n_seeds >= 1 && n_seeds <= (int64_t)n_cu * most &&
           small_walk_group(n_cu, n_seeds) <= most;
}

template <int E>
static hipError_t launch_small_e(hipStream_t stream, int max_lds_bytes, int n_cu, FusedJob f,
                                 SmallScan* ss, hipEvent_t done) {
    const int W = small_walk_group(n_cu, f.n_seeds);
    const int share = (160 * 1024 - 512) / 4 / W & ~3;
    fused_lds_plan(&f, share);
    const size_t lds_bytes = (size_t)W * f.lds_words_per_wave * 4;
    if (f.lds_rows < 1 || lds_bytes + 512 > (size_t)max_lds_bytes) return hipErrorInvalidValue;
    if (lds_bytes > 48 * 1024) {
        hipError_t rc = hipFuncSetAttribute(reinterpret_cast<const void*>(walk_rpe_small_kernel<E>),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (rc != hipSuccess) return rc;
    }
    launch_and_mark(walk_rpe_small_kernel<E>, dim3((unsigned)((f.n_seeds + W - 1) / W)),
                    dim3(W * kWave), lds_bytes, stream, done, f, ss);
    return hipGetLastError();
}

hipError_t launch_walk_rpe_small(hipStream_t stream, int max_lds_bytes, int n_cu,
                                 const int32_t* row_ptr, const int32_t* col_idx, int32_t n_nodes,
                                 int64_t n_edges, const int32_t* seeds, int64_t n_seeds, int32_t M,
                                 int32_t m, uint64_t rng_seed, int32_t* walks, int64_t cap_rows,
                                 int64_t* rpe_off, int32_t* ids, uint16_t* cnt, void* small_scan,
                                 uint32_t spin_limit, int64_t* h_total, hipEvent_t done,
                                 uint32_t* err) {
    const FusedJob f = fused_job(row_ptr, col_idx, n_nodes, n_edges, seeds, n_seeds, M, m, rng_seed,
                                 walks, cap_rows, rpe_off, ids, cnt, EdgeRecords{}, spin_limit,
                                 h_total, err);
    SmallScan* ss = static_cast<SmallScan*>(small_scan);
    const int n_key = fused_keys(M, m);
#define SUREL_WRS_SIZE(E_)            \
    if (n_key <= kWave * (E_))        \
        return launch_small_e<E_>(stream, max_lds_bytes, n_cu, f, ss, done);
    SUREL_FOR_SORT_SIZES(SUREL_WRS_SIZE)
#undef SUREL_WRS_SIZE
    return hipErrorInvalidValue;
}

}  // namespace surel
