// The pieces of the union join (Sec. 3.4, set-union form) that its kernels share: where a query's
// blocks lie, how their id lists are united in LDS, and how the union's rows are written.
//
// A query is worked on by `n_waves` wavefronts: one in the kernels for long query lists (the
// number of queries in flight hides the latency), several in the kernel for short ones (there the
// time of a single query is what counts).  kMulti tells the two apart at compile time.
//
// Uniting.  Two lists by merge path: thread t owns merged positions [t*VT, (t+1)*VT): a binary
// search on its diagonal finds where it starts in both lists, then it merges VT steps serially,
// list 0 first on ties, so an equal pair is one row with two sources.  What the merge leaves
// behind is two bits per union row ("list 0 has this node", "list 1 has it"), kept as two bit
// masks in LDS: both lists are ascending like the union, so the table row of list j that feeds
// union row r is the number of rows before r whose bit j is set, a population count away for the
// lane that handles row r.  Triples are united two lists at a time: the union of lists 0 and 1 is
// written out in LDS (from its masks) and united with list 2 the same way; which of the first two
// lists hold a row of the final union is looked up in the masks of the first merge.  (Before, a
// triple's rows were ranked by binary searches of every node in all other lists.)
//
// Writing.  A lane takes one union row: it gathers the row's K vectors of LT = m + 1 counts from
// the table (zeros where the node is absent) as the aligned words that cover them, packs them into
// the row's words in registers, and the row goes out either straight from the registers (rows of
// whole words that one store takes) or through an LDS tile that is laid out like the output and
// streamed out 16 bytes per lane (join_tiled).  In a filling launch with a large output (kPastBytes in
// join.hip) a query's rounds of 64 rows lie like the output's groups of 32 (the masks start that many bits in), so that all lines of the
// output but a query's first and last are written whole by one instruction, and the stores go past
// the caches: the 1,048,576 pairs of the 2.9M-node graph 5.11 ms, 4.98 with the rounds in place, 4.46
// past the caches as well; 262,144 triples 1.33 -> 1.18, 262,144 pairs of codes 0.80 -> 0.64.  (Rounds
// that are not in place lose past the caches, 6.04 ms: pieces of a line go to memory one by one.)
#pragma once

#include "device_util.h"
#include "lines.h"

namespace surel {

constexpr uint32_t kNoId = 0xFFFFFFFFu;  // no node id reaches 2^28

// Aligned 32-bit words that cover a vector of LT counts wherever it starts.
__host__ __device__ constexpr int join_cover(int LT) { return LT % 2 == 0 ? LT / 2 : LT / 2 + 1; }

// Rounds of 64 union rows whose gathers a wave has in flight together.  More rounds shorten a
// wave's chain of memory round trips but cost registers, i.e. waves per compute unit; the measure is
// the words a lane holds.  Pairs of m = 4: 4.59 ms with four rounds (24 words), 4.46 with six, 4.44
// with eight; triples of m = 3: 1.22 ms with three (18 words), 1.19 with four, 1.18 with five, of m = 2
// 0.87 with four, 1.02 with five; pairs of codes: 0.65 ms with four (8 words), 0.64 with eight and ten.
__host__ __device__ constexpr int join_rounds(int K, int LT, bool past) {
    const int most = K == 3 ? 4 : past && join_cover(LT) == 1 ? 8 : 6;
    const int fit = (K == 2 ? 36 : 27) / (K * join_cover(LT));
    return fit < 1 ? 1 : (fit < most ? fit : most);
}

// Rows go out through an LDS tile, 64 rows and up to 16 bytes in front so that it is aligned like
// the output it goes to, where a lane cannot store its row in one instruction: vectors of an odd
// number of counts, whose rows straddle words, and rows of more than 16 bytes, of which every store
// instruction would write a piece (each line of the output then takes several requests: 30,011
// pairs of m = 9 402 us from the tile, 542 from registers; 262,144 triples of m = 3 1.33 and 1.58 ms).
__host__ __device__ constexpr bool join_tiled(int K, int LT) { return LT % 2 != 0 || K * LT > 8; }
__host__ __device__ constexpr int join_tile_words(int K, int LT) {
    return join_tiled(K, LT) ? (kWave * K * LT + 1) / 2 + 4 : 0;
}

// LDS of one query, in 32-bit words.
struct JoinLds {
    int ids;         // pairs: lists 0 and 1, max_set words each; triples: the same, later list 2
    int u01;         // triples: the union of lists 0 and 1, [2 * max_set]
    int mask01;      // triples: its masks, [2][mask01_words]
    int mask01_words;
    int mask;        // masks of the (final) union, [2][mask_words]
    int mask_words;
    int tile;        // per wave
    int tile_words;
    int total;
};

// One bit per union row, in whole 64-bit words, and two words of slack: a thread's bits are put
// in as three 32-bit words at a time.
__host__ __device__ constexpr int join_mask_words(int rows) { return 2 * ((rows + 63) / 64) + 2; }

__host__ __device__ constexpr JoinLds join_lds_layout(int K, int max_set, int LT, int n_waves) {
    JoinLds o{};
    o.ids = 0;
    int at = 2 * max_set;
    if (K == 3) {
        o.u01 = at;
        at += 2 * max_set;
        o.mask01 = at;
        o.mask01_words = join_mask_words(2 * max_set);
        at += 2 * o.mask01_words;
    }
    o.mask = at;  // even: the masks are read as 64-bit words
    o.mask_words = join_mask_words(kRowsAlign - 1 + K * max_set);
    at += 2 * o.mask_words;
    o.tile_words = join_tile_words(K, LT);
    if (o.tile_words > 0) {
        at = (at + 3) & ~3;
        o.tile_words = (o.tile_words + 3) & ~3;
    }
    o.tile = at;
    at += n_waves * o.tile_words;
    o.total = at;
    return o;
}

// The threads that work on one query.
template <bool kMulti>
struct JoinTeam {
    int lane, wave, n_waves;
    uint32_t* sums;  // kMulti: n_waves words of LDS
    __device__ __forceinline__ int tid() const { return kMulti ? wave * kWave + lane : lane; }
    __device__ __forceinline__ int threads() const { return kMulti ? n_waves * kWave : kWave; }
    __device__ __forceinline__ void sync() const {
        if constexpr (kMulti) {
            __syncthreads();
        } else {
            wave_sync();
        }
    }
    // Exclusive prefix sum of one value per thread; *total = the sum.
    __device__ __forceinline__ int excl_sum(int v, int* total) const {
        const int incl = (int)wave_incl_sum((uint32_t)v);
        if constexpr (!kMulti) {
            *total = (int)wave_bcast_u32((uint32_t)incl, kWave - 1);
            return incl - v;
        } else {
            __syncthreads();  // sums may still be read from the call before
            if (lane == kWave - 1) sums[wave] = (uint32_t)incl;
            __syncthreads();
            int before = 0, sum = 0;
            for (int w = 0; w < n_waves; ++w) {
                if (w < wave) before += (int)sums[w];
                sum += (int)sums[w];
            }
            *total = sum;
            return before + incl - v;
        }
    }
};

// Union size of two lists by merge path, and the two bit masks of the union rows
// (bit first_bit + r of amask: list A holds the node of row r; bmask likewise).  The masks must be zero on
// entry; they are complete after the next team sync.  kLong: a thread may have more than 64 rows
// (the longest triples on one wavefront).
template <bool kMulti, bool kLong = false>
__device__ __forceinline__ int merge_path_union(const uint32_t* A, int nA, const uint32_t* B, int nB,
                                                uint32_t* amask, uint32_t* bmask,
                                                const JoinTeam<kMulti>& team, int first_bit = 0) {
    const int T = nA + nB;
    const int VT = (T + team.threads() - 1) / team.threads();  // at most 64; kLong: 96
    const int d0 = min(team.tid() * VT, T);
    const int d1 = min(d0 + VT, T);
    // split of the first d0 merged elements: a0 from A (ties go to A first), d0 - a0 from B
    int lo = max(0, d0 - nB);
    int hi = min(d0, nA);
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (A[mid] <= B[d0 - 1 - mid]) {
            lo = mid + 1;
        } else {
            hi = mid;
        }
    }
    int a = lo, b = d0 - lo;

    // The thread's VT merge steps.  Every step that takes an A element emits a row; a step that
    // takes a B element emits one unless it equals the last A element taken (the same node: ids
    // are distinct inside a list), which may have been taken by the thread before this one.
    // Only the list that moved is read again.
    int n_emit = 0;
    uint64_t fa = 0, fb = 0;  // bit i: this thread's i-th row has a source in A / in B
    uint64_t fa2 = 0, fb2 = 0;  // kLong: the same for its rows 64 ..
    uint32_t last_a = a > 0 ? A[a - 1] : kNoId;
    uint32_t va = a < nA ? A[a] : kNoId;
    uint32_t vb = b < nB ? B[b] : kNoId;
    for (int d = d0; d < d1; ++d) {
        const bool take_a = (b >= nB) || (a < nA && va <= vb);
        if (take_a) {
            const uint64_t bit = 1ull << (n_emit & 63);
            const bool both = b < nB && vb == va;
            if (!kLong || n_emit < 64) {
                fa |= bit;
                if (both) fb |= bit;
            } else {
                fa2 |= bit;
                if (both) fb2 |= bit;
            }
            n_emit += 1;
            last_a = va;
            a += 1;
        } else {
            if (vb != last_a) {
                const uint64_t bit = 1ull << (n_emit & 63);
                if (!kLong || n_emit < 64) {
                    fb |= bit;
                } else {
                    fb2 |= bit;
                }
                n_emit += 1;
            }
            b += 1;
        }
        const uint32_t* list = take_a ? A : B;
        const int at = take_a ? a : b;
        const bool more = at < (take_a ? nA : nB);
        const uint32_t next = more ? list[at] : kNoId;
        va = take_a ? next : va;
        vb = take_a ? vb : next;
    }
    int n_out;
    const int row0 = first_bit + team.excl_sum(n_emit, &n_out);
    // the thread's rows start at row0: its bits go in there, as up to three 32-bit words
    auto put = [&](uint32_t* mask, uint64_t bits, int first) {
        if (bits == 0ull) return;
        const int w = first >> 5;
        const int sh = first & 31;
        const uint64_t low = bits << sh;
        const uint32_t w0 = (uint32_t)low;
        const uint32_t w1 = (uint32_t)(low >> 32);
        const uint32_t w2 = sh ? (uint32_t)(bits >> (64 - sh)) : 0u;
        if (w0) atomicOr(mask + w, w0);
        if (w1) atomicOr(mask + w + 1, w1);
        if (w2) atomicOr(mask + w + 2, w2);
    };
    put(amask, fa, row0);
    put(bmask, fb, row0);
    if (kLong) {
        put(amask, fa2, row0 + 64);
        put(bmask, fb2, row0 + 64);
    }
    return n_out;
}

// Which of two united lists feed the 64 union rows r0 .. r0+63 (r0 a multiple of 64): lane l
// learns for row r0 + l whether list j feeds it and from which of the list's rows.  before[j] =
// rows of list j that feed union rows below r0; it is moved on to r0 + 64.  An index is checked
// against the list's length, which only a malformed (unsorted) table can exceed.
__device__ __forceinline__ void pair_sources(const uint32_t* mask, int mask_words, int r0, int nA,
                                             int nB, int (&before)[2], int lane, bool (&present)[2],
                                             int (&index)[2]) {
    const int n[2] = {nA, nB};
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const uint64_t bits = *reinterpret_cast<const uint64_t*>(mask + j * mask_words + (r0 >> 5));
        const int rank = (int)__builtin_amdgcn_mbcnt_hi(
            (uint32_t)(bits >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bits, 0u));
        index[j] = before[j] + rank;
        present[j] = ((bits >> lane) & 1ull) != 0ull && index[j] < n[j];
        before[j] += __popcll(bits);
    }
}

// Set bits of a mask below bit n (one wavefront, wave-uniform result).
__device__ __forceinline__ int mask_bits_below(const uint32_t* mask, int n, int lane) {
    int sum = 0;
    for (int t = lane; t * 32 < n; t += kWave) {
        uint32_t w = mask[t];
        if (n - t * 32 < 32) w &= (1u << (n - t * 32)) - 1u;
        sum += __popc(w);
    }
    return (int)wave_bcast_u32(wave_incl_sum((uint32_t)sum), kWave - 1);
}

// The blocks of one query.
template <int K>
struct JoinQuery {
    int64_t lo[K];  // first table row of block j
    int n[K];       // rows of block j
    int n01;        // triples: rows of the union of blocks 0 and 1
};

// Looks the K blocks of query q up (the same in every lane); returns the problem's bits (then the
// query is unusable: it yields no rows).
template <int K>
__device__ __forceinline__ uint32_t join_lookup(int64_t q, const int64_t* __restrict__ rpe_off,
                                                int64_t n_blocks, int32_t max_set,
                                                const int32_t* __restrict__ queries,
                                                JoinQuery<K>& jq) {
    uint32_t problem = 0;
#pragma unroll
    for (int j = 0; j < K; ++j) {
        const int32_t b = queries[q * K + j];
        jq.lo[j] = 0;
        jq.n[j] = 0;
        if (b < 0 || (int64_t)b >= n_blocks) {
            problem |= kDevBadQuery;
        } else {
            const int64_t a = rpe_off[b];
            const int64_t len = rpe_off[b + 1] - a;
            if (a < 0 || len < 0) {
                problem |= kDevBadTable;
            } else if (len > (int64_t)max_set) {
                problem |= kDevSetTooLarge;
            } else {
                jq.lo[j] = a;
                jq.n[j] = (int)len;
            }
        }
    }
    return problem;
}

// Writes the union of lists 0 and 1 (its masks are complete) to u01, 64 rows a time and wave.
template <bool kMulti>
__device__ __forceinline__ void materialize_union(const uint32_t* ids, int max_set, int n0, int n1,
                                                  const uint32_t* mask, int mask_words, int n01,
                                                  uint32_t* u01, const JoinTeam<kMulti>& team) {
    const int rounds = (n01 + kWave - 1) / kWave;
    const int per_wave = kMulti ? (rounds + team.n_waves - 1) / team.n_waves : rounds;
    const int first = kMulti ? team.wave * per_wave : 0;
    const int last = min(first + per_wave, rounds);
    if (first >= last) return;
    int before[2] = {0, 0};
    if (kMulti && first > 0) {
        before[0] = mask_bits_below(mask, first * kWave, team.lane);
        before[1] = mask_bits_below(mask + mask_words, first * kWave, team.lane);
    }
    for (int g = first; g < last; ++g) {
        bool present[2];
        int index[2];
        pair_sources(mask, mask_words, g * kWave, n0, n1, before, team.lane, present, index);
        int at = 0;
        if (present[1]) at = max_set + index[1];
        if (present[0]) at = index[0];
        const int r = g * kWave + team.lane;
        if (r < n01) u01[r] = ids[at];
    }
}

// Unites a query's lists.  `stage(dst, j)` puts list j into LDS at dst (the team's threads
// together; no sync).  The masks that join_write needs are left in LDS.  Returns the
// number of union rows (the same in every thread); the LDS contents are complete after the next
// team sync.
template <int K, bool kMulti, typename Stage>
__device__ __forceinline__ int join_unite(uint32_t* base, const JoinLds& lay, int max_set,
                                          JoinQuery<K>& jq, const JoinTeam<kMulti>& team,
                                          int first_bit, Stage&& stage) {
    uint32_t* ids = base + lay.ids;
    uint32_t* mask = base + lay.mask;
    const int (&n)[K] = jq.n;
    stage(ids, 0);
    stage(ids + max_set, 1);
    for (int t = team.tid(); t < 2 * lay.mask_words; t += team.threads()) mask[t] = 0u;
    if constexpr (K == 2) {
        team.sync();
        return merge_path_union<kMulti>(ids, n[0], ids + max_set, n[1], mask,
                                                mask + lay.mask_words, team, first_bit);
    } else {
        uint32_t* mask01 = base + lay.mask01;
        uint32_t* u01 = base + lay.u01;
        for (int t = team.tid(); t < 2 * lay.mask01_words; t += team.threads()) mask01[t] = 0u;
        team.sync();
        jq.n01 = merge_path_union<kMulti>(ids, n[0], ids + max_set, n[1], mask01,
                                                mask01 + lay.mask01_words, team);
        team.sync();
        materialize_union<kMulti>(ids, max_set, n[0], n[1], mask01, lay.mask01_words, jq.n01, u01,
                                  team);
        team.sync();  // lists 0 and 1 are dead
        stage(ids, 2);
        team.sync();
        if (jq.n01 + n[2] > 64 * team.threads())
            return merge_path_union<kMulti, true>(u01, jq.n01, ids, n[2], mask,
                                                          mask + lay.mask_words, team, first_bit);
        return merge_path_union<kMulti>(u01, jq.n01, ids, n[2], mask,
                                                mask + lay.mask_words, team, first_bit);
    }
}

// Stores past the caches or through them.
template <bool kPast, typename T>
__device__ __forceinline__ void join_store(T* to, T value) {
    if constexpr (kPast) {
        __builtin_nontemporal_store(value, to);
    } else {
        *to = value;
    }
}

// Writes the n_out > 0 union rows of a query that join_unite left in LDS (first_bit as
// there) to rows [off, off + n_out) of the output; wave w of the team takes a contiguous share of
// the rounds.  kPast: they go past the caches (see the file's head).
template <int K, int LT, bool kMulti, bool kPast>
__device__ __forceinline__ void join_write(uint32_t* base, const JoinLds& lay,
                                           const JoinQuery<K>& jq, int first_bit, int n_out,
                                           int64_t off, const uint16_t* __restrict__ rpe_cnt, int max_set,
                                           int32_t* __restrict__ out_ids,
                                           uint16_t* __restrict__ out_cnt, uint16_t absent16,
                                           const JoinTeam<kMulti>& team) {
    constexpr int kCounts = K * LT;             // of a row
    constexpr int kWords = (kCounts + 1) / 2;   // words of a row, packed from its first count
    constexpr int kHalf = LT / 2;               // whole words of a vector
    constexpr int kCover = join_cover(LT);
    constexpr int kRounds = join_rounds(K, LT, kPast);
    const int lane = team.lane;
    const uint32_t* mask = base + lay.mask;
    const uint32_t* mask01 = base + lay.mask01;
    uint32_t* tile32 = base + lay.tile + (kMulti ? team.wave * lay.tile_words : 0);
    const int (&n)[K] = jq.n;
    // the two lists of the last merge
    const uint32_t* ids_a = K == 2 ? base + lay.ids : base + lay.u01;
    const uint32_t* ids_b = K == 2 ? base + lay.ids + max_set : base + lay.ids;
    const int n_a = K == 2 ? n[0] : jq.n01;
    const int n_b = n[K - 1];
    const uint32_t absent32 = (uint32_t)absent16 * 0x10001u;

    // Where list j's vectors are: the aligned word at or before the first of them (uniform), and
    // whether that one starts in the word's upper half.  A lane then gets by with 32-bit
    // arithmetic: its vector starts odd[j] + (row in the list) * LT counts in.  A list without
    // rows has no vectors to point at: the table's first row stands in (the table has rows, or
    // there would be no union rows to write).
    const uint32_t* vec_words[K];
    uint32_t odd[K];
#pragma unroll
    for (int j = 0; j < K; ++j) {
        const uint16_t* first = rpe_cnt + (n[j] > 0 ? jq.lo[j] : 0) * LT;
        odd[j] = LT % 2 == 0 ? 0u : (uint32_t)((reinterpret_cast<uintptr_t>(first) >> 1) & 1u);
        vec_words[j] = reinterpret_cast<const uint32_t*>(first - odd[j]);
    }

    // Rows are counted from the first bit of the masks on.
    out_ids += off - first_bit;
    out_cnt += (off - first_bit) * kCounts;
    int r_first = 0, r_last = first_bit + n_out;
    int before[2] = {0, 0};     // rows of the two merged lists below the present round
    int before01[2] = {0, 0};   // triples: rows of lists 0 and 1 below it
    if constexpr (kMulti) {
        const int rounds = (r_last + kWave - 1) / kWave;
        const int per_wave = (rounds + team.n_waves - 1) / team.n_waves;
        r_first = team.wave * per_wave * kWave;
        r_last = min(r_first + per_wave * kWave, r_last);
        if (r_first >= r_last) return;
        if (r_first > 0) {
            before[0] = mask_bits_below(mask, r_first, lane);
            before[1] = mask_bits_below(mask + lay.mask_words, r_first, lane);
            if constexpr (K == 3) {
                before01[0] = mask_bits_below(mask01, before[0], lane);
                before01[1] = mask_bits_below(mask01 + lay.mask01_words, before[0], lane);
            }
        }
    }
    // kRounds rounds of 64 rows are gathered together (all their loads are in flight before the
    // first is waited for: a wave's time is a chain of memory round trips), then the rounds go
    // out one after the other
    for (int r0 = r_first; r0 < r_last; r0 += kRounds * kWave) {
        uint32_t raw[kRounds][K][kCover + 1];
        uint32_t shift[kRounds][K];
        bool present[kRounds][K];
        uint32_t id[kRounds];
        if constexpr (kPast) {  // below, rounds past the last row are waited for with the others
#pragma unroll
            for (int g = 0; g < kRounds; ++g)
#pragma unroll
                for (int j = 0; j < K; ++j)
#pragma unroll
                    for (int t = 0; t < kCover; ++t) raw[g][j][t] = any_value();
        }
#pragma unroll
        for (int g = 0; g < kRounds; ++g) {
            if (r0 + g * kWave >= r_last) break;  // wave-uniform: no round past the last row
            bool in[2];
            int at[2];
            pair_sources(mask, lay.mask_words, r0 + g * kWave, n_a, n_b, before, lane, in, at);
            // the node's id, from the first list that has it (a lane past the last row reads the
            // first id and stores nothing)
            const uint32_t* from = in[0] ? ids_a + at[0] : ids_b + (in[1] ? at[1] : 0);
            id[g] = *from;
            int index[K];
            if constexpr (K == 2) {
                present[g][0] = in[0], present[g][1] = in[1];
                index[0] = at[0], index[1] = at[1];
            } else {
                present[g][2] = in[1];
                index[2] = at[1];
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int p = in[0] ? at[0] : 0;
                    const uint32_t word = mask01[j * lay.mask01_words + (p >> 5)];
                    const bool has = in[0] && ((word >> (p & 31)) & 1u) != 0u;
                    const uint64_t all = __ballot(has);
                    index[j] = before01[j] + (int)__builtin_amdgcn_mbcnt_hi(
                        (uint32_t)(all >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)all, 0u));
                    present[g][j] = has && index[j] < n[j];
                    before01[j] += __popcll(all);
                }
            }
#pragma unroll
            for (int j = 0; j < K; ++j) {
                // unconditional loads, from the list's first row where it has no row for the
                // node: a branch would make every load wait for the one before it.  A vector is
                // read as the aligned words that cover it (misaligned wide loads are taken apart
                // lane by lane by the L1) and shifted into place afterwards; the last word may
                // reach one count past the vector, never past the word that holds the table's
                // last count.
                const uint32_t first = odd[j] + (uint32_t)(present[g][j] ? index[j] : 0) * LT;
                shift[g][j] = (first & 1u) * 2u;
                const uint32_t* aligned = vec_words[j] + (first >> 1);
#pragma unroll
                for (int t = 0; t < kCover; ++t) raw[g][j][t] = aligned[t];
                raw[g][j][kCover] = 0u;
            }
        }
        // All of them are waited for here: in the middle of stores past the caches, every wait for a load
        // would wait for stores as well (pairs of codes 0.80 -> 0.72 ms).  Stores that the caches take
        // are soon done, and the rounds better go out as their vectors come (20,000 pairs 98 -> 80 us).
#pragma unroll
        for (int g = 0; g < kRounds; ++g)
#pragma unroll
            for (int j = 0; j < K; ++j)
#pragma unroll
                for (int t = 0; t < kCover; ++t)
                    if constexpr (kPast) asm volatile("" : "+v"(raw[g][j][t]));
#pragma unroll
        for (int g = 0; g < kRounds; ++g) {
            if (r0 + g * kWave >= r_last) break;
            // word t of vector j holds its counts 2t and 2t+1; a vector of an odd number of
            // counts ends in the low half of its last word
            uint32_t w[kWords + 1];
            w[kWords] = 0u;
#pragma unroll
            for (int j = 0; j < K; ++j) {
                uint32_t vec[kCover];
#pragma unroll
                for (int t = 0; t < kCover; ++t) {
                    vec[t] = LT % 2 == 0 ? raw[g][j][t]
                                         : __builtin_amdgcn_alignbyte(raw[g][j][t + 1], raw[g][j][t],
                                                                      shift[g][j]);
                    if (!present[g][j]) vec[t] = absent32;
                }
                const int start = j * LT;  // first count of the vector inside the row
                if (start % 2 == 0) {
#pragma unroll
                    for (int t = 0; t < kHalf; ++t) w[start / 2 + t] = vec[t];
                    if (LT % 2 == 1) w[start / 2 + kHalf] = vec[kHalf] & 0xFFFFu;
                } else {
                    w[(start - 1) / 2] |= vec[0] << 16;
#pragma unroll
                    for (int t = 0; t < kHalf; ++t)
                        w[(start + 1) / 2 + t] = __builtin_amdgcn_alignbyte(vec[t + 1], vec[t], 2u);
                }
            }
            const int r1 = r0 + g * kWave;
            const int r = r1 + lane;
            const bool live = (!kPast || r >= first_bit) && r < r_last;
            if (live) join_store<kPast>(out_ids + r, (int32_t)id[g]);
            if constexpr (!join_tiled(K, LT)) {
                // a lane's row is stored from its registers, in one instruction: the rows of
                // neighbouring lanes adjoin, so a wave's store is contiguous
                if (live) {
                    typedef uint32_t row_t __attribute__((ext_vector_type(kWords), aligned(4)));
                    row_t row;
#pragma unroll
                    for (int d = 0; d < kWords; ++d) row[d] = w[d];
                    uint32_t* row_words = reinterpret_cast<uint32_t*>(out_cnt) + (int64_t)r * kWords;
                    row_t* to = reinterpret_cast<row_t*>(row_words);
                    if constexpr (kPast) {
                        __builtin_nontemporal_store(row, to);
                    } else {
                        *to = row;
                    }
                }
            } else {
                // The rows are put together in an LDS tile and go out 16 bytes per lane.  The tile
                // starts `head` counts in, so that 16-byte pieces of the tile are 16-byte pieces of
                // the output.
                uint16_t* dst = out_cnt + (int64_t)r1 * kCounts;
                const int head = (int)((reinterpret_cast<uintptr_t>(dst) >> 1) & 7u);
                uint16_t* tile16 = reinterpret_cast<uint16_t*>(tile32);
                if constexpr (kCounts % 2 == 0) {  // pairs: rows of whole words (head is even)
#pragma unroll
                    for (int d = 0; d < kWords; ++d) tile32[(head >> 1) + lane * kWords + d] = w[d];
                } else {
                    // triples: every other row starts in the middle of a word; a lane writes the
                    // whole words inside its row and the half word at its end or its start
                    const int p = head + lane * kCounts;
                    const bool mid = (p & 1) != 0;
                    uint32_t* words = tile32 + ((p + 1) >> 1);
#pragma unroll
                    for (int d = 0; d + 1 < kWords; ++d)
                        words[d] = __builtin_amdgcn_alignbyte(w[d + 1], w[d], mid ? 2u : 0u);
                    tile16[mid ? p : p + kCounts - 1] = (uint16_t)(mid ? w[0] : w[kWords - 1]);
                }
                wave_sync();
                constexpr int kUnit = kCounts % 2 == 0 ? 2 : 1;  // counts moved at a time at the ends
                // counts [first, last) of the tile are rows; the 16-byte pieces that lie in there
                // are [lead, tail)
                const int first = kPast ? max(first_bit - r1, 0) * kCounts : 0;
                const int last = min(r_last - r1, kWave) * kCounts;
                const int lead = min(((head + first + 7) & ~7) - head, last);
                const int n_quads = (last - lead) >> 3;
                const int tail = lead + 8 * n_quads;
                typedef uint32_t quad_t __attribute__((ext_vector_type(4)));
                const quad_t* tile_quads = reinterpret_cast<const quad_t*>(tile16 + head + lead);
                quad_t* dst_quads = reinterpret_cast<quad_t*>(dst + lead);
                if constexpr (kUnit == 2) {
                    const uint32_t* t32 = tile32 + (head >> 1);
                    uint32_t* d32 = reinterpret_cast<uint32_t*>(dst);
                    if (lane < (lead - first) / 2) d32[first / 2 + lane] = t32[first / 2 + lane];
                    for (int t = lane; t < n_quads; t += kWave)
                        join_store<kPast>(dst_quads + t, tile_quads[t]);
                    if (lane < (last - tail) / 2) d32[tail / 2 + lane] = t32[tail / 2 + lane];
                } else {
                    if (lane < lead - first) dst[first + lane] = tile16[head + first + lane];
                    for (int t = lane; t < n_quads; t += kWave)
                        join_store<kPast>(dst_quads + t, tile_quads[t]);
                    if (lane < last - tail) dst[tail + lane] = tile16[head + tail + lane];
                }
                wave_sync();
            }
        }
    }
}

}  // namespace surel
