// From a wave's sorted walk keys to the rows of one seed's RPE block (Sec. 3.2 "Relative
// Positional Encoding"): a key is node id << 4 | walk position; id changes start rows, and every
// key adds to the count of its (row, position).  Shared by the stand-alone RPE builder and the
// fused walk + RPE kernels.
#pragma once

#include "device_util.h"

namespace surel {

// Keys that fill the sort up to 64*E: an id no node has, so they sort last and form one row of
// their own behind the block's rows.  Their 16 position values keep them from all counting in the
// same LDS word.
constexpr uint32_t kPadKeys = 0xFFFFFFF0u;
__device__ __forceinline__ uint32_t pad_key(int lane) { return kPadKeys | ((uint32_t)lane & 15u); }

// Walk keys of a wave: the sort is compiled for these numbers of keys per lane.  (Vector instructions of a
// sort, wave_sort.h: 482 with 7, 518 with 8, 670 with 9, 734 with 10, 874 with 12, 1,050 with 13, 1,090 with
// 14, 1,182 with 16; 15 and 11 take no fewer than 16 and 12.  Walks + RPE of 235,000 seeds of M = 200, m = 4,
// 801 keys: 1,361 us with 16, 1,298 with 13; of 99,991 of M = 61, m = 9, 550 keys: 493 with 10, 483 with 9;
// walks of 2.9M-node graphs wait for memory and take the same time.)
#define SUREL_FOR_SORT_SIZES(X) \
    X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(12) X(13) X(14) X(16) X(20) X(24) X(32)

template <int E>
__device__ __forceinline__ void copy_keys(uint32_t (&to)[E], const uint32_t (&from)[E]) {
    to[0] = from[0];
    if constexpr (E > 1) {
#pragma unroll
        for (int r = 1; r < E; ++r) to[r] = from[r];
    }
}

// What a lane knows about the rows of the wave's sorted keys (sort position p = lane*E + r).
struct RpeRowScan {
    uint32_t before;     // key just before this lane's first
    int32_t first_row;   // row of that key (-1 in lane 0)
    int32_t n_rows;      // rows of the whole wave (wave-uniform), the padding's not counted
};

template <int E>
__device__ __forceinline__ RpeRowScan rpe_scan_rows(const uint32_t (&x)[E], int lane) {
    RpeRowScan sc;
    sc.before = wave_from_lane_below(x[E - 1]);
    if (lane == 0) sc.before = ~x[0];  // the first key starts a row
    uint32_t n_head = 0;
    uint32_t prev = sc.before;
#pragma unroll
    for (int r = 0; r < E; ++r) {
        n_head += (x[r] ^ prev) > 15u ? 1u : 0u;
        prev = x[r];
    }
    const uint32_t incl = wave_incl_sum(n_head);
    sc.first_row = (int32_t)(incl - n_head) - 1;
    const bool padded = (uint32_t)__builtin_amdgcn_readlane((int)x[E - 1], kWave - 1) >= kPadKeys;
    sc.n_rows = (int32_t)wave_bcast_u32(incl, kWave - 1) - (padded ? 1 : 0);
    return sc;
}

// LDS words that hold up to `rows` rows of a block: ids (behind up to three words that align them
// like their destination), then counts (behind up to seven counts), each with room for the
// padding's row.
__host__ __device__ constexpr int rpe_id_words(int rows) { return (rows + 1 + 3 + 3) & ~3; }
__host__ __device__ constexpr int rpe_cnt_words(int rows, int L) {
    return (rows * L + 16 + 7 + 1 + 7) / 8 * 4;
}
__host__ __device__ constexpr int rpe_row_words(int rows, int L) {
    return rpe_id_words(rows) + rpe_cnt_words(rows, L);
}

// Assembles rows [row0, row0 + n) of the block in LDS: ids[0 .. n) and counts cnt16[0 .. n*L).
// cnt_words: the 16-byte aligned words that hold cnt16, which starts `head` counts in; they are
// cleared here.  The key of position 0, if `start_weight` is not 0, stands for that many walks
// that start at its node.  Ends with the LDS writes ordered before later reads.
// No lane is ever masked out: every key of a row writes the row's id, a key's count is an
// addition in LDS (no runs of equal keys to be found), and the rows outside the window, like the
// padding's, all go to the row behind it.
template <int E>
__device__ __forceinline__ void rpe_assemble_rows(const uint32_t (&x)[E], const RpeRowScan& sc,
                                                  int lane, int L, int row0, int n,
                                                  uint32_t start_weight, uint32_t* ids,
                                                  uint32_t* cnt_words, int head) {
    uint4* clear = reinterpret_cast<uint4*>(cnt_words);
    for (int t = lane; t * 8 < head + n * L; t += kWave) clear[t] = make_uint4(0u, 0u, 0u, 0u);
    wave_sync();
    uint32_t prev = sc.before;
    int32_t row = sc.first_row - row0;
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const uint32_t key = x[r];
        row += (key ^ prev) > 15u ? 1 : 0;
        prev = key;
        const uint32_t to = min((uint32_t)row, (uint32_t)n);
        const uint32_t pos = key & 15u;
        const uint32_t weight = start_weight != 0u && pos == 0u ? start_weight : 1u;
        const uint32_t at = (uint32_t)head + (uint32_t)__umul24(to, (uint32_t)L) + pos;
        ids[to] = key >> 4;
        atomicAdd(cnt_words + (at >> 1), weight << ((at & 1u) * 16u));
    }
    wave_sync();
}

// Moves n 32-bit words, or 16-bit counts, from LDS to global memory, 16 bytes per
// lane where it can: src lies at the same place inside a 16-byte piece as dst.  past: past the caches.
// kFew: what one instruction takes goes out a value a lane: a piece and its two ends would be three (walks +
// RPE of 2 M seeds of M = 5, m = 4 3,396 -> 3,333 us, 2.9 M tables of M = 20, m = 2 1,023 -> 955).  Blocks of
// that kind have up to 128 keys; longer ones are not asked for it.
constexpr bool few_values(int E) { return E <= 2; }  // E: sort keys per lane
template <bool kFew, typename T>
__device__ __forceinline__ void stream_aligned(const T* src, T* __restrict__ dst, int n, int lane,
                                               bool past) {
    constexpr int kPer = 16 / (int)sizeof(T);
    const int head = (int)((reinterpret_cast<uintptr_t>(dst) / sizeof(T)) & (kPer - 1));
    const int lead = kFew && n <= kWave ? n : min((kPer - head) & (kPer - 1), n);
    const int n_quads = (n - lead) / kPer;
    const int tail = lead + n_quads * kPer;
    if (lane < lead) dst[lane] = src[lane];
    typedef uint32_t quad_t __attribute__((ext_vector_type(4)));
    const quad_t* s4 = reinterpret_cast<const quad_t*>(src + lead);
    quad_t* d4 = reinterpret_cast<quad_t*>(dst + lead);
    if (past) {
        for (int t = lane; t < n_quads; t += kWave) __builtin_nontemporal_store(s4[t], d4 + t);
    } else {
        for (int t = lane; t < n_quads; t += kWave) d4[t] = s4[t];
    }
    if (lane < n - tail) dst[tail + lane] = src[tail + lane];
}

// Whether a table's rows go past the caches: where it may take twice the 256 MB memory-side cache, of
// which a half to two thirds come out.  Then the rows only push the records out of the L2s that walks
// keep there (walks + table of 235,000 seeds of M = 200, m = 4: 1.58 -> 1.55 ms; 500,009 tables of
// M = 50, m = 4 from finished walks: 423 -> 403 us).  A smaller table is still there when a join reads
// it (20,000 pairs of M = 100, m = 4 on 30,000 nodes 83 us, 100 when the table went past the caches).
inline bool table_goes_past(int64_t n_seeds, int32_t M, int32_t m) {
    return n_seeds * (1 + (int64_t)M * m) * (4 + 2 * (m + 1)) > (int64_t)512 << 20;
}

// Writes the block's rows to rows [off, off + sc.n_rows) of the table, at most lds_rows of them
// at a time (lds: rpe_row_words(lds_rows, L) words, 16-byte aligned; blocks that need more than
// one turn are rare, the LDS of a wave decides how many waves a compute unit holds).  cnt may be
// null: a table that carries RPE-IDs only.  each(row0, n, cnt16, free_words) is called for every
// turn while its counts lie in LDS (from cnt16 on), with n words of LDS that are free again.
template <int E, typename Each>
__device__ __forceinline__ void rpe_write_rows(const uint32_t (&x)[E], const RpeRowScan& sc,
                                               int lane, int L, uint32_t start_weight,
                                               uint32_t* lds, int lds_rows, int64_t off,
                                               int32_t* __restrict__ ids,
                                               uint16_t* __restrict__ cnt, bool past, Each&& each) {
    uint32_t* cnt_words = lds + rpe_id_words(lds_rows);
    for (int row0 = 0; row0 < sc.n_rows; row0 += lds_rows) {
        const int n = min(lds_rows, sc.n_rows - row0);
        int32_t* dst_ids = ids + off + row0;
        uint16_t* dst_cnt = cnt == nullptr ? nullptr : cnt + (off + row0) * L;
        uint32_t* lds_ids = lds + (int)((reinterpret_cast<uintptr_t>(dst_ids) >> 2) & 3u);
        const int head = (int)((reinterpret_cast<uintptr_t>(dst_cnt) >> 1) & 7u);
        rpe_assemble_rows<E>(x, sc, lane, L, row0, n, start_weight, lds_ids, cnt_words, head);
        const uint16_t* cnt16 = reinterpret_cast<const uint16_t*>(cnt_words) + head;
        stream_aligned<few_values(E)>(reinterpret_cast<const int32_t*>(lds_ids), dst_ids, n, lane, past);
        wave_sync();
        each(row0, n, cnt16, lds_ids);
        if (cnt != nullptr) stream_aligned<few_values(E)>(cnt16, dst_cnt, n * L, lane, past);
        wave_sync();  // the LDS words are free again
    }
}

}  // namespace surel
