// What the two fused walk + RPE kernels do with one seed: walk it into an LDS block, send the
// block out, turn it into sort keys and sort them (Sec. 3.2: the RPE is computed on the fly as the
// walks get sampled).
#pragma once

#include "device_util.h"
#include "kernels.h"
#include "rpe_rows.h"
#include "walk_core.h"
#include "wave_sort.h"

namespace surel {

constexpr int kFusedChains = 2;  // walks a lane moves at a time

// Sort keys of a seed: every step of every walk, and ONE key for the M walks' common start
// (sorting M equal keys would be work for nothing: 1,000 keys instead of 801 at M = 200, m = 4).
__host__ __device__ constexpr int fused_keys(int M, int m) { return M * m + 1; }
// LDS words of the walk block: M rows of m + 1 positions, a scratch row for the idle lanes of the last
// pass, and up to three words in front.
__host__ __device__ constexpr int fused_block_words(int M, int m) {
    return ((M + 1) * (m + 1) + 3 + 3) & ~3;
}

struct FusedJob {
    WalkGraph g;
    const int32_t* __restrict__ seeds;
    int64_t n_seeds;
    int32_t M, m;
    uint32_t key0, key1;  // of the random stream
    uint32_t magic_m;     // 65536 / m + 1, see small_div
    int32_t* __restrict__ walks;
    int64_t cap_rows;
    int64_t* __restrict__ rpe_off;
    int32_t* __restrict__ ids;
    uint16_t* __restrict__ cnt;
    int32_t lds_words_per_wave;
    int32_t lds_rows;     // rows of a block that fit there at a time
    bool past;            // the table's rows go past the caches
    uint32_t spin_limit;
    int64_t* h_total;     // host memory that gets the row total too, or null
    uint32_t* __restrict__ err;
};

// Lays out the LDS of a wave that may have `share` words: the walk block, or as many rows of an RPE
// block as fit (a block with more rows goes out in turns); lds_rows = 0: not even one fits.
inline void fused_lds_plan(FusedJob* f, int share) {
    const int L = f->m + 1;
    const int block_words = fused_block_words(f->M, f->m);
    const int room = share > block_words ? share : block_words;
    f->lds_rows = 1 + f->M * f->m;  // App. D.4: at most m*M nodes besides the seed
    while (f->lds_rows > 0 && rpe_row_words(f->lds_rows, L) > room) f->lds_rows -= 1;
    const int row_words = (rpe_row_words(f->lds_rows, L) + 3) & ~3;
    f->lds_words_per_wave = row_words > block_words ? row_words : block_words;
}

inline FusedJob fused_job(const int32_t* row_ptr, const int32_t* col_idx, int32_t n_nodes,
                          int64_t n_edges, const int32_t* seeds, int64_t n_seeds, int32_t M,
                          int32_t m, uint64_t rng_seed, int32_t* walks, int64_t cap_rows,
                          int64_t* rpe_off, int32_t* ids, uint16_t* cnt, const EdgeRecords& rec,
                          uint32_t spin_limit, int64_t* h_total, uint32_t* err) {
    return FusedJob{{row_ptr, col_idx, rec.data, rec.id_bits, rec.lo_bits, n_nodes, n_edges},
                    seeds, n_seeds, M, m, (uint32_t)(rng_seed & 0xFFFFFFFFull),
                    (uint32_t)(rng_seed >> 32), 65536u / (uint32_t)m + 1u, walks, cap_rows, rpe_off,
                    ids, cnt, 0, 0, table_goes_past(n_seeds, M, m), spin_limit, h_total, err};
}

// Writes -1 for all walks of seed number i, which is not a node.
__device__ __forceinline__ void fused_bad_seed(const FusedJob& f, int64_t i, int lane) {
    const int n = f.M * (f.m + 1);
    int32_t* out = f.walks + i * (int64_t)n;
    if (lane == 0) atomicOr(f.err, kDevBadSeed);
    for (int t = lane; t < n; t += kWave) __builtin_nontemporal_store(-1, out + t);
}

// Walks seed number i (node u) and leaves its sorted keys in y.  block: LDS of the wave, dead
// afterwards.
template <int E, int kRec>
__device__ __forceinline__ void fused_walk_and_sort(const FusedJob& f, int64_t i, int32_t u,
                                                    int32_t* block, int lane, uint32_t (&y)[E]) {
    const int M = f.M, m = f.m, L = m + 1;
    // it lies in LDS at the same place inside a 16-byte piece as in its output
    int32_t* out = f.walks + i * (int64_t)(M * L);
    block += (reinterpret_cast<uintptr_t>(out) >> 2) & 3u;
    int32_t u_lo, u_deg;
    bool bad_graph = seed_row(f.g, u, &u_lo, &u_deg);
    for (int w0 = 0; w0 < M; w0 += kFusedChains * kWave) {
        int w[kFusedChains];
        bool active[kFusedChains];
        int32_t* row[kFusedChains];
#pragma unroll
        for (int c = 0; c < kFusedChains; ++c) {
            w[c] = w0 + c * kWave + lane;
            active[c] = w[c] < M;
            // lanes past the last walk share one scratch row behind the block
            row[c] = block + (active[c] ? w[c] : M) * L;
        }
        if (w0 + kWave < M) {
            bad_graph |= walk_many<kRec, kFusedChains>(f.g, u, u_lo, u_deg, w, active, m, f.key0,
                                                       f.key1, row, [](int, int32_t) {});
        } else {  // one walk a lane is left
            const int w1[1] = {w[0]};
            const bool active1[1] = {active[0]};
            int32_t* const row1[1] = {row[0]};
            bad_graph |= walk_many<kRec, 1, false>(f.g, u, u_lo, u_deg, w1, active1, m, f.key0, f.key1, row1,
                                            [](int, int32_t) {});
        }
    }
    raise_error(f.err, bad_graph, kDevBadGraph);
    wave_sync();
    // the block goes out as it lies in LDS
    stream_aligned<few_values(E)>(block, out, M * L, lane, true);
    // Keys: entry idx of the steps is step 1 + idx mod m of walk idx / m.  A register's entries lie
    // 64 behind those of the register before it.  (Worked out anew for every seed, which the asm
    // makes the compiler believe: kept over the seeds, the places of all E registers are 2E
    // registers, which are waves.)
    const uint32_t n_step = (uint32_t)(M * m);
    uint32_t idx = (uint32_t)lane;
    asm volatile("" : "+v"(idx));
    const uint32_t walk = small_div(idx, f.magic_m);
    uint32_t pos = idx - walk * (uint32_t)m;
    uint32_t at = idx + walk + 1u;
    const uint32_t next_walk = small_div(kWave, f.magic_m);
    const uint32_t next_pos = kWave - next_walk * (uint32_t)m;
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const uint32_t v = (uint32_t)block[min(at, n_step + (uint32_t)M - 1u)];
        const uint32_t key = (v << 4) | (pos + 1u);
        y[r] = idx < n_step ? key : (idx == n_step ? (uint32_t)u << 4 : pad_key(lane));
        const bool wraps = pos + next_pos >= (uint32_t)m;
        pos = wraps ? pos + next_pos - (uint32_t)m : pos + next_pos;
        at += kWave + next_walk + (wraps ? 1u : 0u);
        idx += kWave;
    }
    wave_sync();  // the walk block in LDS is dead from here on
    wave_sort<E>(y, lane);
}

}  // namespace surel
