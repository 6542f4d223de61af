// Pruning the central RPE array (Sec. 3.3; Algorithm 1, last step): many table rows carry the
// same count vector, so the distinct vectors are stored once, in an array T, and every row
// keeps the index of its vector in T (its RPE-ID after re-indexing).  The paper leaves T in
// insertion order; here T is sorted (count vectors compared entry by entry), which makes the
// result unique and testable bit for bit.
//
// Steps, all on the device:
//   collect  every row looks its vector up in a global open-addressing hash set and inserts it if
//            it is new (prune_set.h); the vector's number in the set goes to the codes.  A slot is
//            64 bytes (state, number, vector), aligned, so one cache line holds all of it; only a
//            slot that does not look full yet is touched with atomics.
//   rank     every vector's place in the sorted array: up to prune_rank_most vectors are compared
//            all with all (a few thousand, usually: one short launch that needs no count on the
//            host), more are sorted with a bitonic network in global memory.
//   codes    code[row] = place of the row's vector, from the numbers (which are 16 bits each where no
//            larger ones occur, see kNarrowMost).
//            The launch stores T as well, and empties the slots that were used again, by the list of the
//            set's members (a memset of the table, and a pass over it that gathers the full slots,
//            were 95 us of a call with cap_T = 2^20).  With so many vectors that the slots are still
//            asked then, they are emptied behind it.
// Waiting.  A lane that finds a slot locked (another lane is writing its vector) polls it
// again; the writer needs nothing from the poller (inside one wavefront the writer's branch
// runs to its end before the next poll), so the poll ends; it is bounded by the spin limit
// all the same.
#include <cmath>
#include <type_traits>

#include "device_util.h"
#include "kernels.h"
#include "lines.h"
#include "prune_set.h"

namespace surel {

constexpr int kTableWords = kDirectWords + CollectTables::kHashed;
constexpr int kWarmRows = 2 * kWave;
// Rows of a wave's tile, the list of rows that wait for a look-up, and wavefronts of a workgroup,
// which share the LDS tables (32 KB): as many as its LDS then holds.
template <int LT>
struct Collect {
    static constexpr int kRows = LT == 0 ? 128 : 512;
    static constexpr int kMaxL = LT == 0 ? 16 : LT;
    static constexpr int kTileWords = kRows * kMaxL / 2;
    static constexpr int kQuads = (kTileWords / 4 + kWave - 1) / kWave;  // 16-byte pieces a lane moves
    static constexpr int kMisses = LT == 0 ? 0 : kRows;         // of half a word each
    static constexpr int kLate = LT == 0 ? 0 : 2 * kWave;       // of four words each
    static constexpr int kWaveWords = kTileWords + kMisses / 2 + 4 * kLate;
    static constexpr int kFit = (160 * 1024 / 4 - kTableWords) / kWaveWords;
    static constexpr int kWaves = kFit < 16 ? kFit : 16;
};

// Numbers of a tile on their way to the renumbering.  While a wave has seen no number above kNarrowMost, its
// tiles' numbers go out in 16 bits, in the first half of the tile's codes: a lane's rows (g * kWave + lane) * 2
// and the one behind, g = 0 .. 3, are the 16 bytes at lane * 16, and kNarrowMost + 1 is a row whose vector the
// renumbering looks up once more (one that was on the late list and has a larger number).  From then on a tile
// is its codes as they stand, with kWide set in each, so that any word of a tile tells which of both it is.
// (Numbers are handed out in the order of insertion, so the commonest vectors have small ones.)
// 146 M rows of 1M seeds with 1,500 vectors are pruned in 522 us, 692 with numbers of 32 bits and other
// ways to the caches; 60 M with 100,000 vectors, nearly all of them wide, in 1.90 ms, 1.98.
constexpr int32_t kNarrowMost = 0x7FFE;
constexpr uint32_t kNarrowUnknown = (uint32_t)kNarrowMost + 1u;
constexpr uint32_t kWide = 0x80000000u;
// place of a row of a tile among the 16-bit numbers
__device__ __forceinline__ int narrow_place(int t) {
    return ((t >> 1) & (kWave - 1)) * 8 + (t / (2 * kWave)) * 2 + (t & 1);
}

// Rows whose vectors no LDS table has, with their vectors (as pairs of counts, see row_pairs): looked
// up in the global table together once there are 64 of them, for the look-up is a chain of trips to
// memory behind the counts on their way.
template <int LT>
struct LateList {
    static constexpr int NW = (LT + 1) / 2;
    static constexpr int kRoom = Collect<LT>::kLate;
    uint4* items;  // pairs 0 .. NW-1, row
    int n;
    uint32_t wide_from;  // the first row of the wave's that went out wide (~0: none yet)
    __device__ __forceinline__ void append(uint64_t all, bool mine, const uint32_t (&pair)[NW], uint32_t row) {
        const int before = (int)__builtin_amdgcn_mbcnt_hi(
            (uint32_t)(all >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)all, 0u));
        if (mine)
            items[n + before] = make_uint4(pair[0], NW > 1 ? pair[NW > 1 ? 1 : 0] : 0u,
                                           NW > 2 ? pair[NW > 2 ? 2 : 0] : 0u, row);
        n += __popcll(all);
    }
    // tile(row): the codes of the row's tile.  next: the first row that has not gone out yet.
    template <typename Tile>
    __device__ __forceinline__ void resolve(int lane, uint32_t next, uint32_t* cache,
                                            const VectorSet& set, Tile&& tile) {
        constexpr uint32_t kRows = Collect<LT>::kRows;
        const uint32_t wide_before = wide_from;
        wave_sync();
        for (int u0 = 0; u0 < n; u0 += kWave) {
            const bool valid = u0 + lane < n;
            const uint4 item = items[valid ? u0 + lane : 0];
            const uint32_t all[3] = {item.x, item.y, item.z};
            uint32_t pair[NW], w[NW], at;
#pragma unroll
            for (int k = 0; k < NW; ++k) {
                pair[k] = all[k];
                w[k] = (all[k] << 16) | (all[k] >> 16);
            }
            const bool small = DirectIndex<LT>::of(pair, &at);
            const int32_t number = lookup_hashed<NW, CollectTables>(w, hash_vector<NW>(w), valid,
                                                                     cache + kDirectWords, set, lane);
            if (valid && small && number >= 0) cache[at] = (uint32_t)number + 1u;
            if (wide_from == ~0u && __ballot(valid && number > kNarrowMost) != 0ull) wide_from = next;
            if (valid) {
                int32_t* codes = tile(item.w);
                const int t = (int)(item.w % kRows);
                if (item.w >= wide_before) {
                    codes[t] = (int32_t)((uint32_t)number | kWide);
                } else if ((uint32_t)number < kNarrowUnknown) {
                    reinterpret_cast<uint16_t*>(codes)[narrow_place(t)] = (uint16_t)number;
                }
            }
        }
        n = 0;
        wave_sync();
    }
};

// The numbers of the rows of a whole tile, two neighbouring rows a lane: they are LT whole words, so
// the places of their counts are known at compile time.  Rows that the direct table does not have are
// put on a list (misses) and looked up in the hashed cache; their numbers come back through the tile,
// whose rows are dead then, so that the codes go out in whole lines.  Only rows that the cache does not
// have either go on the list `late`, and out a second time when that is resolved (while it has room;
// else the global table is asked at once).  first: number of the tile's first row there.
// (With all rows that the direct table does not have on the late list, two in a hundred went out a
// second time to a line that had left the caches: 2.6 M more writes beside 9.1 M, a fifth of the time.
// With none on it, tables with many vectors waited for the global table in every tile.)
template <int LT>
__device__ __forceinline__ void tile_numbers(uint32_t* tile, int lane, uint32_t first, uint16_t* misses,
                                             LateList<LT>& late, uint32_t* cache, const VectorSet& set,
                                             int32_t* __restrict__ code) {
    constexpr int NW = (LT + 1) / 2;
    constexpr int kRows = Collect<LT>::kRows;
    constexpr int kTurns = kRows / (2 * kWave);
    int32_t number[kTurns][2];
    uint64_t missed[kTurns][2];
    int n_miss = 0;
#pragma unroll
    for (int g = 0; g < kTurns; ++g) {
        const int t = (g * kWave + lane) * 2;
        const uint32_t* from = tile + (t / 2) * LT;
        uint32_t raw[LT];
#pragma unroll
        for (int k = 0; k < LT; ++k) raw[k] = from[k];
        uint32_t pair[2][NW];
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            if constexpr (LT % 2 == 0) {
                pair[0][k] = raw[k];
                pair[1][k] = raw[NW + k];
            } else {
                pair[0][k] = k + 1 < NW ? raw[k] : raw[k] & 0xFFFFu;
                pair[1][k] = k + 1 < NW ? __builtin_amdgcn_alignbyte(raw[NW + k], raw[NW - 1 + k], 2u)
                                        : raw[LT - 1] >> 16;
            }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint32_t at;
            const bool small = DirectIndex<LT>::of(pair[h], &at);
            const uint32_t e = cache[at];
            number[g][h] = (int32_t)(e - 1u);
            missed[g][h] = __ballot(!(small && e != 0u));
            append_misses(misses, n_miss, !(small && e != 0u), t + h);
        }
    }
    uint16_t* tile16 = reinterpret_cast<uint16_t*>(tile);
    if (n_miss > 0) {
        wave_sync();
        for (int u0 = 0; u0 < n_miss; u0 += kWave) {
            const bool valid = u0 + lane < n_miss;
            const int t = (int)misses[valid ? u0 + lane : 0];
            uint32_t pair[NW], w[NW], at;
            row_pairs<NW>(tile, 0, kRows * LT / 2, t, LT, pair);
            const bool small = DirectIndex<LT>::of(pair, &at);
#pragma unroll
            for (int k = 0; k < NW; ++k) w[k] = (pair[k] << 16) | (pair[k] >> 16);
            const uint32_t hv = hash_vector<NW>(w);
            int32_t found = cached_number<NW, CollectTables>(w, hv, cache + kDirectWords);
            const bool unknown = valid && found < 0;
            const uint64_t all = __ballot(unknown);
            if (all != 0ull) {
                if (late.n + __popcll(all) <= LateList<LT>::kRoom) {
                    late.append(all, unknown, pair, first + (uint32_t)t);
                } else {
                    found = lookup_hashed<NW, CollectTables>(w, hv, valid, cache + kDirectWords, set, lane);
                }
            }
            if (valid && small && found >= 0) cache[at] = (uint32_t)found + 1u;
            if (valid) {
                tile16[t * LT] = (uint16_t)(uint32_t)found;
                tile16[t * LT + 1] = (uint16_t)((uint32_t)found >> 16);
            }
        }
        wave_sync();
#pragma unroll
        for (int g = 0; g < kTurns; ++g) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (missed[g][h] == 0ull) continue;
                const uint16_t* row = tile16 + ((g * kWave + lane) * 2 + h) * LT;
                const uint32_t found = (uint32_t)row[0] | (uint32_t)row[1] << 16;
                number[g][h] = ((missed[g][h] >> lane) & 1ull) != 0ull ? (int32_t)found : number[g][h];
            }
        }
    }
    if (late.wide_from == ~0u) {
        bool large = false;
#pragma unroll
        for (int g = 0; g < kTurns; ++g) large = large || max(number[g][0], number[g][1]) > kNarrowMost;
        if (__ballot(large) != 0ull) late.wide_from = first;
    }
    if (late.wide_from == ~0u) {
        static_assert(kTurns == 4, "a lane's rows are 16 bytes");
        typedef uint32_t quad_t __attribute__((ext_vector_type(4), aligned(4)));
        quad_t all;
#pragma unroll
        for (int g = 0; g < kTurns; ++g)
            all[g] = min((uint32_t)number[g][0], kNarrowUnknown) | min((uint32_t)number[g][1], kNarrowUnknown) << 16;
        reinterpret_cast<quad_t*>(code)[lane] = all;
        return;
    }
    typedef uint32_t two_t __attribute__((ext_vector_type(2), aligned(4)));
#pragma unroll
    for (int g = 0; g < kTurns; ++g) {
        const two_t both = {(uint32_t)number[g][0] | kWide, (uint32_t)number[g][1] | kWide};
        reinterpret_cast<two_t*>(code)[g * kWave + lane] = both;
    }
}

// A wavefront takes tiles of consecutive rows: they come in as contiguous 16-byte pieces (the next
// tile's are on their way while one is looked up) and are read row by row from LDS.
// What bounds it: the stream of counts in and numbers out, and the chain of a tile through LDS.  146 M rows
// of 1M seeds with some 1,500 vectors 344 us = 5.1 TB/s.  The counts go past the caches and the numbers do not
// (both past them 378 us, counts through them 386; the renumbering then finds more of the numbers: 146 us, 166
// where they went past; 60 M rows pruned in 578 us, 586 where they went past, 700 M 6.09 ms and 6.07).  Two
// tiles ahead: 355 us where one took 343.  The tile's loads and the numbers' stores are in one straight
// line, so that a wait for the next tile is not one for the numbers.
template <int LT>
__global__ __launch_bounds__(Collect<LT>::kWaves* kWave) void prune_collect_kernel(
    const uint16_t* __restrict__ cnt, int64_t n_rows, int L, int32_t* __restrict__ code,
    VectorSet set) {
    using C = Collect<LT>;
    constexpr int kRows = C::kRows, kQuads = C::kQuads;
    extern __shared__ __align__(16) uint32_t lds32[];
    uint32_t* cache = lds32;
    set_cache_clear(cache, kTableWords, (int)threadIdx.x, C::kWaves * kWave);
    __syncthreads();
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    uint32_t* tile = lds32 + kTableWords + wave * C::kWaveWords;
    const int n_quads = kRows * L / 8;  // whole 16-byte pieces
    typedef uint32_t quad_t __attribute__((ext_vector_type(4), aligned(4)));  // the array is 4-byte aligned
    const int64_t stride = (int64_t)gridDim.x * C::kWaves;
    const int64_t n_whole = n_rows / kRows;
    int64_t at = (int64_t)blockIdx.x * C::kWaves + wave;
    quad_t next[kQuads];
    auto fetch = [&](int64_t t) {
        const quad_t* from = reinterpret_cast<const quad_t*>(cnt + t * kRows * L);
#pragma unroll
        for (int u = 0; u < kQuads; ++u)
            if (LT > 0 || u * kWave + lane < n_quads) next[u] = __builtin_nontemporal_load(from + u * kWave + lane);
    };
    auto to_lds = [&]() {
        uint4* to = reinterpret_cast<uint4*>(tile);
#pragma unroll
        for (int u = 0; u < kQuads; ++u)
            if (LT > 0 || u * kWave + lane < n_quads)
                to[u * kWave + lane] = make_uint4(next[u][0], next[u][1], next[u][2], next[u][3]);
        wave_sync();
    };
    uint16_t* misses = reinterpret_cast<uint16_t*>(tile + C::kTileWords);
    LateList<LT == 0 ? 2 : LT> late{reinterpret_cast<uint4*>(tile + C::kTileWords + C::kMisses / 2), 0, ~0u};
    // a wave's rows are numbered along its own tiles, so that 32 bits do for a table of any size
    const int64_t at0 = at;
    uint32_t first = 0;
    auto tile_of = [&](uint32_t row) -> int32_t* {
        return code + (at0 + (int64_t)(row / kRows) * stride) * kRows;
    };
    if (at < n_whole) {
        fetch(at);
        to_lds();
    }
    // the first wave's first tile on its own: it fills the workgroup's tables with the common
    // vectors, for which the other waves then need not ask the global table all at once
    for (int turn = 0; turn < 2; ++turn) {
        if (turn == 1) __syncthreads();
        while (at < n_whole && (turn == 1 || wave == 0)) {
            int32_t* out = code + at * kRows;
            at += stride;
            if (at < n_whole) fetch(at);
            if constexpr (LT > 0) {
                // before anything is known all rows of a tile would go on the list: a few make most
                // of the others known (what they leave in the tile's codes is written over)
                if (turn == 0) {
                    rows_numbers<LT, CollectTables>(kWarmRows, lane, L, reinterpret_cast<const uint16_t*>(tile),
                                                     misses, cache, set, out);
                    wait_memory();
                }
                tile_numbers<LT>(tile, lane, first, misses, late, cache, set, out);
                if (late.n >= kWave) late.resolve(lane, first + kRows, cache, set, tile_of);
            } else {
                rows_numbers<0, CollectTables>(kRows, lane, L, reinterpret_cast<const uint16_t*>(tile),
                                                nullptr, cache, set, out);
            }
            first += kRows;
            wave_sync();
            if (at < n_whole) to_lds();
            if (turn == 0) break;
        }
        if constexpr (LT > 0) late.resolve(lane, first, cache, set, tile_of);
    }
    // the rows behind the last whole tile
    const int rest = (int)(n_rows - n_whole * kRows);
    if (at == n_whole && rest > 0) {
        uint16_t* tile16 = reinterpret_cast<uint16_t*>(tile);
        for (int t = lane; t < rest * L; t += kWave) tile16[t] = cnt[n_whole * kRows * L + t];
        wave_sync();
        rows_numbers<LT, CollectTables>(rest, lane, L, tile16, misses, cache, set, code + n_whole * kRows);
    }
}

// Vectors are compared all with all up to so many word comparisons (n^2 times the words of a
// vector): about 0.09 ns a thousand, so 0.45 ms, which is what the sort's launches take for this many
// vectors (one compare-exchange launch of 3 to 4 us for every step, 105 to 136 of them).  The whole
// pruning of 4 M rows, all pairs against the sort, in us (differences are the ranking's):
//   vectors          16,384        32,768         65,536
//   1 word         256 / 586     357 / 654      662 /   813
//   3 words        426 / 712     649 / 789    1,463 /   933
//   8 words        779 / 954   1,353 / 1,046  3,528 / 1,178
// so the line lies at 70,710, 40,824 and 25,000 vectors of 1, 3 and 8 words.
constexpr int64_t kRankWords = 5'000'000'000;
constexpr int kRankTile = 256;
constexpr int kRankBlocks = 1024;
// Up to so many vectors a tile is compared with a quarter of another at a time: still a workgroup each, and
// the launch takes as long as one workgroup's loop (1,500 vectors of three words 11.7 -> 5.0 us).
constexpr int kRankFew = 4096;

// ranks[i] += vectors of one tile that are smaller than vector i of another, for all pairs of
// tiles.  The number of vectors is read on the device, so that the launch does not wait for the
// host to learn it; with more of them than this launch is for, it does nothing.
template <int NW>
__global__ __launch_bounds__(kRankTile) void prune_rank_pairs_kernel(
    const uint32_t* __restrict__ members, const unsigned long long* __restrict__ n_inserted,
    int64_t most, uint32_t* __restrict__ ranks) {
    __shared__ uint32_t other[NW][kRankTile];
    const int64_t n = (int64_t)*n_inserted;
    if (n > most) return;
    const int64_t tiles = (n + kRankTile - 1) / kRankTile;
    const int width = n <= kRankFew ? kRankTile / 4 : kRankTile;
    const int64_t parts = (n + width - 1) / width;
    for (int64_t p = blockIdx.x; p < tiles * parts; p += gridDim.x) {
        const int64_t i = (p / parts) * kRankTile + threadIdx.x;
        const int64_t j0 = (p % parts) * width;
        uint32_t mine[NW];
#pragma unroll
        for (int k = 0; k < NW; ++k) mine[k] = i < n ? members[i * kItemWords + k] : 0u;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NW; ++k)
            other[k][threadIdx.x] = j0 + threadIdx.x < n ? members[(j0 + threadIdx.x) * kItemWords + k] : ~0u;
        __syncthreads();
        const int m = (int)min((int64_t)width, n - j0);
        uint32_t smaller = 0;
        for (int j = 0; j < m; ++j) {
            bool less = false;
#pragma unroll
            for (int k = NW - 1; k >= 0; --k)
                less = other[k][j] < mine[k] || (other[k][j] == mine[k] && less);
            smaller += less ? 1u : 0u;
        }
        if (i < n && smaller != 0u) atomicAdd(&ranks[i], smaller);
    }
}

// What the launch that renumbers the codes does besides (RankedSet::finish, called by all its threads with
// the number of vectors): T[ranks[i]] = vector i; with up to clean_most vectors the slots of the set's
// members are emptied; the counters of the call after this one are cleared (two calls take turns with two
// sets of them, so nobody has to know who reads the present ones last); the number of vectors also goes to
// host memory, and whether a wait ran out.  (As launches of their own, with a clearing of the counters by
// their last workgroup, T and the slots took 5 + 4 us and the gaps before them; with the ranks, above,
// 250,000 rows with 1,500 vectors are pruned in 74 us instead of 85.)
struct RankedSet {
    const uint32_t* __restrict__ members;
    const unsigned long long* __restrict__ counters;
    unsigned long long* next_counters;
    const uint32_t* __restrict__ ranks;
    uint32_t* slots;
    uint16_t* T;
    int64_t most, clean_most;
    int L;
    int64_t* h_n_T;
    int64_t* h_stalled;
    __device__ __forceinline__ void finish(int64_t n) const {
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            *h_n_T = n;
            if (counters[2] != 0ull) *h_stalled = 1;
            next_counters[0] = 0ull;
            next_counters[2] = 0ull;
        }
        if (n > most) return;
        for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
             i += (int64_t)gridDim.x * blockDim.x) {
            const uint32_t* item = members + i * kItemWords;
            const int64_t place = ranks[i];
            for (int e = 0; e < L; ++e) {
                const uint32_t word = item[e >> 1];
                T[place * L + e] = (uint16_t)((e & 1) ? (word & 0xFFFFu) : (word >> 16));
            }
            if (n <= clean_most) slots[(size_t)item[kMaxVecWords] * kSlotWords] = kSlotEmpty;
        }
    }
};

// Empties the slots of the set's members.
__global__ __launch_bounds__(256) void prune_clean_kernel(const uint32_t* __restrict__ members,
                                                          int64_t n, uint32_t* __restrict__ slots) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) slots[(size_t)members[i * kItemWords + kMaxVecWords] * kSlotWords] = kSlotEmpty;
}

// Entries from `first` on become padding that sorts behind every vector.
__global__ __launch_bounds__(256) void prune_pad_kernel(uint32_t* __restrict__ list, int64_t first,
                                                        int64_t len) {
    const int64_t i = first + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= len) return;
#pragma unroll
    for (int k = 0; k <= kMaxVecWords; ++k) list[i * kItemWords + k] = 0xFFFFFFFFu;
}

__device__ __forceinline__ bool item_less(const uint32_t (&a)[kMaxVecWords + 1],
                                          const uint32_t (&b)[kMaxVecWords + 1]) {
#pragma unroll
    for (int k = 0; k <= kMaxVecWords; ++k) {
        if (a[k] != b[k]) return a[k] < b[k];
    }
    return false;
}

// One compare-exchange step of a bitonic sorting network over `len` (a power of two) items:
// partner distance j inside merges of size k.
__global__ __launch_bounds__(256) void prune_sort_step_kernel(uint32_t* __restrict__ list,
                                                              int64_t len, int64_t j, int64_t k) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t p = i ^ j;
    if (i >= len || p <= i) return;
    uint32_t a[kMaxVecWords + 1], b[kMaxVecWords + 1];
#pragma unroll
    for (int t = 0; t <= kMaxVecWords; ++t) {
        a[t] = list[i * kItemWords + t];
        b[t] = list[p * kItemWords + t];
    }
    const bool ascending = (i & k) == 0;
    if (item_less(b, a) == ascending) {
#pragma unroll
        for (int t = 0; t <= kMaxVecWords; ++t) {
            list[i * kItemWords + t] = b[t];
            list[p * kItemWords + t] = a[t];
        }
    }
}

// T[i] = vector of the i-th item of the sorted list, whose number learns its place.
__global__ __launch_bounds__(256) void prune_rank_kernel(const uint32_t* __restrict__ list,
                                                         int64_t n_T, int L,
                                                         const uint32_t* __restrict__ slots,
                                                         uint32_t* __restrict__ ranks,
                                                         uint16_t* __restrict__ T) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_T) return;
    const uint32_t* item = list + i * kItemWords;
    ranks[slots[(size_t)item[kMaxVecWords] * kSlotWords + kSlotNumber]] = (uint32_t)i;
    for (int e = 0; e < L; ++e) {
        const uint32_t word = item[e >> 1];
        T[i * L + e] = (uint16_t)((e & 1) ? (word & 0xFFFFu) : (word >> 16));
    }
}

// code[row]: number of the row's vector -> its place (what is no number becomes -1).
// Four rows a lane, moved as 16-byte words where the array's alignment allows (the pass is a
// plain stream over the codes; the places come from a few thousand words).
// rows (optional): where the number of rows stands on the device (more than cap_rows of them: the
// codes are not all there and stay as they are); n_known < 0: the number of vectors stands in the set's
// counters, with more than set.most the codes stay as they are, and set.finish is called.
constexpr int kCodesUnroll = 4;
__global__ __launch_bounds__(256) void prune_codes_kernel(
    RankedSet set, int64_t n_known, int64_t n_rows, const int64_t* __restrict__ rows,
    int64_t cap_rows, int32_t* __restrict__ code) {
    const uint32_t* __restrict__ ranks = set.ranks;
    const int64_t n = n_known >= 0 ? n_known : (int64_t)set.counters[0];
    if (n_known < 0) set.finish(n);
    if (n > set.most) return;
    if (rows != nullptr) n_rows = *rows;
    if (n_rows > cap_rows) return;
    auto rank_of = [&](int32_t c) -> int32_t {
        return (uint64_t)(uint32_t)c < (uint64_t)n ? (int32_t)ranks[(uint32_t)c] : -1;
    };
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if ((reinterpret_cast<uintptr_t>(code) & 15u) == 0) {
        // kCodesUnroll 16-byte words of a lane are in flight together, past the caches on their way in:
        // every code is read once and written once (then, see codes_go_past)
        typedef int code4_t __attribute__((ext_vector_type(4)));
        code4_t* code4 = reinterpret_cast<code4_t*>(code);
        const int64_t n4 = n_rows / 4;
        auto all = [&](auto past) {  // two loops: with a branch at every store 167 M rows took 35 us longer
            for (int64_t i0 = tid; i0 < n4; i0 += stride * kCodesUnroll) {
                code4_t c[kCodesUnroll];
#pragma unroll
                for (int u = 0; u < kCodesUnroll; ++u) {
                    const int64_t i = i0 + u * stride;
                    c[u] = code4_t{-1, -1, -1, -1};
                    if (i < n4) c[u] = __builtin_nontemporal_load(code4 + i);
                }
#pragma unroll
                for (int u = 0; u < kCodesUnroll; ++u) {
                    const int64_t i = i0 + u * stride;
                    c[u].x = rank_of(c[u].x);
                    c[u].y = rank_of(c[u].y);
                    c[u].z = rank_of(c[u].z);
                    c[u].w = rank_of(c[u].w);
                    if (i >= n4) continue;
                    if constexpr (decltype(past)::value) {
                        __builtin_nontemporal_store(c[u], code4 + i);
                    } else {
                        code4[i] = c[u];
                    }
                }
            }
        };
        if (codes_go_past(n_rows)) {
            all(std::true_type{});
        } else {
            all(std::false_type{});
        }
        for (int64_t row = n4 * 4 + tid; row < n_rows; row += stride) code[row] = rank_of(code[row]);
    } else {
        for (int64_t row = tid; row < n_rows; row += stride) code[row] = rank_of(code[row]);
    }
}

// The same for numbers as the collecting launch leaves them (Collect<LT>, LT > 0): whole tiles narrow or
// wide, then plain numbers.  A wave takes tiles, kCodesUnroll of them in flight; with no more vectors than
// narrow numbers no tile is wide and only the first half of its codes is read.  The first kHotRanks places,
// which nearly all rows have, are in LDS.
// What bounds it: the stream of numbers in and codes out, 0.88 GB of 146 M rows in 146 us = 6 TB/s (from
// numbers of 32 bits 210 us); 8 M rows are bound by the trips before it.
constexpr int kHotRanks = 4096;
template <int LT>
__global__ __launch_bounds__(256) void prune_tile_codes_kernel(
    RankedSet set, int64_t n_known, int64_t n_rows, const uint16_t* __restrict__ cnt,
    uint32_t slot_mask, int32_t* __restrict__ code) {
    const uint32_t* __restrict__ ranks = set.ranks;
    const uint32_t* slots = set.slots;
    constexpr int kRows = Collect<LT>::kRows, NW = (LT + 1) / 2;
    typedef uint32_t quad_t __attribute__((ext_vector_type(4), aligned(4)));
    typedef uint32_t two_t __attribute__((ext_vector_type(2), aligned(4)));
    __shared__ uint32_t hot[kHotRanks];
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t n_whole = n_rows / kRows;
    const int64_t stride = (int64_t)gridDim.x * 4;
    int64_t t0 = (int64_t)blockIdx.x * 4 + wave;
    quad_t low[kCodesUnroll], high[kCodesUnroll];
    auto part = [&](int u) {
        return reinterpret_cast<const quad_t*>(code + min(t0 + u * stride, n_whole - 1) * kRows) + lane;
    };
    auto load_low = [&]() {
#pragma unroll
        for (int u = 0; u < kCodesUnroll; ++u) low[u] = __builtin_nontemporal_load(part(u));
    };
    if (t0 < n_whole) load_low();  // before the trips for the number of vectors and their places
    const int64_t n = n_known >= 0 ? n_known : (int64_t)set.counters[0];
    if (n_known < 0) set.finish(n);
    if (n > set.most) return;
    // (a wave with one tile would wait for this table longer than for its places: 2 M rows 86 -> 85 us)
    const uint32_t n_hot = n_whole > stride ? (uint32_t)min(n, (int64_t)kHotRanks) : 0u;
    if (n_hot != 0u) {
        uint32_t mine[kHotRanks / 256];  // their loads are one trip
#pragma unroll
        for (int u = 0; u < kHotRanks / 256; ++u) {
            const uint32_t t = u * 256 + threadIdx.x;
            mine[u] = t < n_hot ? ranks[t] : 0u;
        }
#pragma unroll
        for (int u = 0; u < kHotRanks / 256; ++u) hot[u * 256 + threadIdx.x] = mine[u];
        __syncthreads();
    }
    auto rank_of = [&](uint32_t c) -> uint32_t {
        return c < n_hot ? hot[c] : c < (uint32_t)n ? ranks[c] : ~0u;
    };
    // a row whose number did not fit: its vector's slot is full and behind no empty one
    auto number_of = [&](int64_t row) -> uint32_t {
        uint32_t w[NW];
#pragma unroll
        for (int k = 0; k < NW; ++k)
            w[k] = (uint32_t)cnt[row * LT + 2 * k] << 16 | (2 * k + 1 < LT ? (uint32_t)cnt[row * LT + min(2 * k + 1, LT - 1)] : 0u);
        uint32_t h = hash_vector<NW>(w) & slot_mask;
        for (uint32_t probe = 0; probe <= slot_mask; ++probe) {
            const uint32_t* slot = slots + (size_t)h * kSlotWords;
            const uint32_t st = slot[0];
            if ((st & kSlotFull) == 0u) break;
            bool same = true;
#pragma unroll
            for (int k = 0; k < NW; ++k) same = same && slot[kSlotVector + k] == w[k];
            if (same) return st & ~kSlotFull;
            h = (h + 1u) & slot_mask;
        }
        return ~0u;
    };
    const bool none_wide = n <= (int64_t)kNarrowMost + 1;
    while (t0 < n_whole) {
        if (!none_wide) {
#pragma unroll
            for (int u = 0; u < kCodesUnroll; ++u) high[u] = __builtin_nontemporal_load(part(u) + kWave);
        }
#pragma unroll
        for (int u = 0; u < kCodesUnroll; ++u) {
            const int64_t t = t0 + u * stride;
            if (t >= n_whole) break;
            int32_t* to = code + t * kRows;
            if (!none_wide && (__builtin_amdgcn_readfirstlane((int)low[u][0]) < 0)) {
                quad_t a, b;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    a[k] = rank_of(low[u][k] & ~kWide);
                    b[k] = rank_of(high[u][k] & ~kWide);
                }
                __builtin_nontemporal_store(a, reinterpret_cast<quad_t*>(to) + lane);
                __builtin_nontemporal_store(b, reinterpret_cast<quad_t*>(to) + kWave + lane);
                continue;
            }
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                uint32_t c[2] = {low[u][g] & 0xFFFFu, low[u][g] >> 16};
                if (!none_wide) {
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        if (c[h] == kNarrowUnknown) c[h] = number_of(t * kRows + (g * kWave + lane) * 2 + h);
                }
                const two_t both = {rank_of(c[0]), rank_of(c[1])};
                __builtin_nontemporal_store(both, reinterpret_cast<two_t*>(to) + g * kWave + lane);
            }
        }
        t0 += stride * kCodesUnroll;
        if (t0 < n_whole) load_low();
    }
    // rows behind the last whole tile: fewer than a tile's
    if (blockIdx.x == gridDim.x - 1) {
        for (int64_t row = n_whole * kRows + threadIdx.x; row < n_rows; row += blockDim.x)
            code[row] = (int32_t)rank_of((uint32_t)code[row]);
    }
}

int64_t prune_slots(int64_t cap_T) {
    int64_t s = 1024;
    while (s < 4 * cap_T) s *= 2;
    return s;
}
int64_t prune_list_len(int64_t cap_T) {
    int64_t s = 1;
    while (s < cap_T) s *= 2;
    return s;
}
size_t prune_slot_bytes(int64_t cap_T) { return (size_t)prune_slots(cap_T) * kSlotWords * 4; }
size_t prune_member_bytes(int64_t cap_T) { return (size_t)prune_list_len(cap_T) * kItemWords * 4; }
size_t prune_rank_bytes(int64_t cap_T) { return (size_t)cap_T * sizeof(uint32_t); }

VectorSet vector_set(const PruneScratch& ps, uint32_t spin_limit, uint32_t* err) {
    return VectorSet{ps.slots, (uint32_t)(prune_slots(ps.cap_T) - 1), ps.cap_T, ps.members, ps.ranks,
                     ps.counters, spin_limit, err};
}

hipError_t launch_prune_clear(hipStream_t stream, const PruneScratch& ps) {
    // (the calls that use the set wait for the host in any case, so they cannot be captured into a
    // graph, and plain memsets do)
    hipError_t rc = hipMemsetAsync(ps.slots, 0, prune_slot_bytes(ps.cap_T), stream);
    if (rc != hipSuccess) return rc;
    rc = hipMemsetAsync(ps.counters, 0, 3 * sizeof(unsigned long long), stream);
    if (rc != hipSuccess) return rc;
    return hipMemsetAsync(ps.next_counters, 0, 3 * sizeof(unsigned long long), stream);
}

template <int LT>
static hipError_t launch_collect(hipStream_t stream, int n_cu, const uint16_t* cnt, int64_t n_rows,
                                 int L, int32_t* code, const VectorSet& set) {
    using C = Collect<LT>;
    const size_t lds_bytes = (size_t)(kTableWords + C::kWaves * C::kWaveWords) * 4;
    const auto kernel = prune_collect_kernel<LT>;
    hipError_t rc = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
    if (rc != hipSuccess) return rc;
    // a workgroup fills its LDS tables once and keeps them
    int64_t blocks = (n_rows / C::kRows + C::kWaves) / C::kWaves;
    if (blocks > n_cu) blocks = n_cu;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(C::kWaves * kWave), lds_bytes, stream, cnt,
                       n_rows, L, code, set);
    return hipGetLastError();
}

hipError_t launch_prune_collect(hipStream_t stream, int n_cu, const uint16_t* cnt, int64_t n_rows,
                                int32_t m, const PruneScratch& ps, int32_t* code,
                                uint32_t spin_limit, uint32_t* err) {
    if (n_rows == 0) return hipSuccess;
    const VectorSet set = vector_set(ps, spin_limit, err);
    const int L = m + 1;
    switch (L) {
        case 2: return launch_collect<2>(stream, n_cu, cnt, n_rows, L, code, set);
        case 3: return launch_collect<3>(stream, n_cu, cnt, n_rows, L, code, set);
        case 4: return launch_collect<4>(stream, n_cu, cnt, n_rows, L, code, set);
        case 5: return launch_collect<5>(stream, n_cu, cnt, n_rows, L, code, set);
        case 6: return launch_collect<6>(stream, n_cu, cnt, n_rows, L, code, set);
        default: return launch_collect<0>(stream, n_cu, cnt, n_rows, L, code, set);
    }
}

template <int LT>
static void launch_tile_codes(hipStream_t stream, int n_cu, const PruneScratch& ps, const RankedSet& set,
                              int64_t n_known, int64_t n_rows, const uint16_t* cnt, int32_t* code) {
    int64_t blocks = n_rows / Collect<LT>::kRows / 4 + 1;
    if (blocks > (int64_t)n_cu * 8) blocks = (int64_t)n_cu * 8;
    hipLaunchKernelGGL(prune_tile_codes_kernel<LT>, dim3((unsigned)blocks), dim3(256), 0, stream, set,
                       n_known, n_rows, cnt, (uint32_t)(prune_slots(ps.cap_T) - 1), code);
}

// Whether the numbers of the collecting launch are tiles of the two forms (Collect<LT>, LT > 0).
static bool numbers_in_tiles(const uint16_t* cnt, int32_t m) { return cnt != nullptr && m <= 5; }

// cnt: the rows' vectors where the numbers come from launch_prune_collect, else null.
static void launch_codes(hipStream_t stream, int n_cu, const PruneScratch& ps, const RankedSet& set,
                         int64_t n_known, int64_t n_rows, const int64_t* d_rows, int64_t cap_rows,
                         const uint16_t* cnt, int32_t* code) {
    if (numbers_in_tiles(cnt, set.L - 1)) {
        switch (set.L) {
            case 2: return launch_tile_codes<2>(stream, n_cu, ps, set, n_known, n_rows, cnt, code);
            case 3: return launch_tile_codes<3>(stream, n_cu, ps, set, n_known, n_rows, cnt, code);
            case 4: return launch_tile_codes<4>(stream, n_cu, ps, set, n_known, n_rows, cnt, code);
            case 5: return launch_tile_codes<5>(stream, n_cu, ps, set, n_known, n_rows, cnt, code);
            default: return launch_tile_codes<6>(stream, n_cu, ps, set, n_known, n_rows, cnt, code);
        }
    }
    int64_t blocks = ((d_rows ? cap_rows : n_rows) / 4 + 256) / 256;
    if (blocks > (int64_t)n_cu * 32) blocks = (int64_t)n_cu * 32;
    hipLaunchKernelGGL(prune_codes_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, set, n_known,
                       n_rows, d_rows, cap_rows, code);
}

int64_t prune_rank_most(int64_t cap_T, int32_t m) {
    const int64_t words = (m + 2) / 2;
    int64_t n = (int64_t)std::sqrt((double)kRankWords / (double)words);
    while (n * n * words > kRankWords) --n;
    return cap_T < n ? cap_T : n;
}

int64_t prune_clean_most(int64_t cap_T, int32_t m, const uint16_t* cnt) {
    // wide tiles' renumbering looks into the slots
    const int64_t most = prune_rank_most(cap_T, m);
    return numbers_in_tiles(cnt, m) && most > (int64_t)kNarrowMost + 1 ? (int64_t)kNarrowMost + 1 : most;
}

hipError_t launch_prune_order(hipStream_t stream, int n_cu, const PruneScratch& ps, int32_t m,
                              int64_t n_rows, const int64_t* d_rows, int64_t cap_rows,
                              const uint16_t* cnt, uint16_t* T, int32_t* code, int64_t* h_n_T,
                              int64_t* h_stalled) {
    const int64_t most = prune_rank_most(ps.cap_T, m);
    const int L = m + 1;
    switch ((L + 1) / 2) {
#define SUREL_RANK_CASE(NW_)                                                                     \
    case NW_:                                                                                    \
        hipLaunchKernelGGL((prune_rank_pairs_kernel<NW_>), dim3(kRankBlocks), dim3(kRankTile), 0, \
                           stream, ps.members, ps.counters, most, ps.ranks);                     \
        break;
        SUREL_RANK_CASE(1)
        SUREL_RANK_CASE(2)
        SUREL_RANK_CASE(3)
        SUREL_RANK_CASE(4)
        SUREL_RANK_CASE(5)
        SUREL_RANK_CASE(6)
        SUREL_RANK_CASE(7)
        SUREL_RANK_CASE(8)
#undef SUREL_RANK_CASE
        default: return hipErrorInvalidValue;
    }
    const RankedSet set{ps.members, ps.counters, ps.next_counters, ps.ranks, ps.slots, T, most,
                        prune_clean_most(ps.cap_T, m, cnt), L, h_n_T, h_stalled};
    launch_codes(stream, n_cu, ps, set, -1, n_rows, d_rows, cap_rows, cnt, code);
    return hipGetLastError();
}

hipError_t launch_prune_clean(hipStream_t stream, const PruneScratch& ps, int64_t n_T) {
    hipLaunchKernelGGL(prune_clean_kernel, dim3((unsigned)((n_T + 255) / 256)), dim3(256), 0, stream,
                       ps.members, n_T, ps.slots);
    return hipGetLastError();
}

hipError_t launch_prune_order_many(hipStream_t stream, int n_cu, const PruneScratch& ps, int32_t m,
                                   int64_t n_rows, int64_t n_T, const uint16_t* cnt, uint16_t* T,
                                   int32_t* code) {
    int64_t len = 1;
    while (len < n_T) len *= 2;  // <= prune_list_len(cap_T) because n_T <= cap_T
    if (len > n_T)
        hipLaunchKernelGGL(prune_pad_kernel, dim3((unsigned)((len - n_T + 255) / 256)), dim3(256), 0,
                           stream, ps.members, n_T, len);
    for (int64_t k = 2; k <= len; k *= 2)
        for (int64_t j = k / 2; j >= 1; j /= 2)
            hipLaunchKernelGGL(prune_sort_step_kernel, dim3((unsigned)((len + 255) / 256)),
                               dim3(256), 0, stream, ps.members, len, j, k);
    hipLaunchKernelGGL(prune_rank_kernel, dim3((unsigned)((n_T + 255) / 256)), dim3(256), 0, stream,
                       ps.members, n_T, m + 1, ps.slots, ps.ranks, T);
    const RankedSet set{ps.members, ps.counters, ps.next_counters, ps.ranks, ps.slots, T, n_T, 0, m + 1,
                        nullptr, nullptr};
    launch_codes(stream, n_cu, ps, set, n_T, n_rows, nullptr, n_rows, cnt, code);
    return hipGetLastError();
}

}  // namespace surel
