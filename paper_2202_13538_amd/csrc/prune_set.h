// The hash set of distinct count vectors behind the pruning of the central RPE array (Sec. 3.3;
// Algorithm 1, last step), shared by the stand-alone pruning kernels and the fused walk + RPE
// kernel when it emits RPE-IDs: a global open-addressing table of 64-byte slots (state with number,
// vector in one cache line) with small per-workgroup tables in LDS in front of it.  A vector is NW
// 32-bit words, entry 2k of the count vector in the upper half of word k, so that comparing words
// in order compares the counts in order.  The vectors of the set are numbered in the order in
// which they are inserted; a vector's number is what a row is given until the numbers become
// places in the sorted array T.
#pragma once

#include "device_util.h"
#include "kernels.h"

namespace surel {

// 64-byte slots: [0] state (empty, locked, or full with the vector's number), [1..8] vector, [9] the
// number once more, which stays when the slot is emptied.  A vector of up to three words is found with
// ONE load of 16 bytes: a look-up is one trip to memory, not three (state, vector, number).
constexpr uint32_t kSlotEmpty = 0u, kSlotLocked = 1u, kSlotFull = 0x80000000u;
constexpr int kSlotWords = 16;
constexpr int kSlotVector = 1;
constexpr int kSlotNumber = kSlotVector + 8;
constexpr int kMaxVecWords = 8;   // m + 1 <= 16 counts of 16 bits
constexpr int kItemWords = kMaxVecWords + 1;  // a member of the set: its vector, zeros, its slot

// The set.  members[i] = vector number i and its slot (kItemWords words; i < cap_T), ranks[i] = 0:
// written by whoever inserts it.  counters[0] = vectors inserted so far; counters[2] becomes 1 if a
// wait runs out.
struct VectorSet {
    uint32_t* slots;
    uint32_t slot_mask;
    int64_t cap_T;
    uint32_t* members;
    uint32_t* ranks;
    unsigned long long* counters;
    uint32_t spin_limit;
    uint32_t* err;
};

VectorSet vector_set(const PruneScratch& ps, uint32_t spin_limit, uint32_t* err);

template <int NW>
__device__ __forceinline__ uint32_t hash_vector(const uint32_t (&w)[NW]) {
    uint32_t h = 0x811C9DC5u;
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        h = (h ^ w[k]) * 0x9E3779B1u;
        h ^= h >> 15;
    }
    return h;
}

// Finds (or inserts) vector w, first probe at slot h; returns its number, or -1 if a wait ran out
// or the table is full.
template <int NW>
__device__ __forceinline__ int32_t find_or_insert(const uint32_t (&w)[NW], uint32_t h,
                                                  const VectorSet& set) {
    uint32_t spins = 0;
    for (uint32_t probe = 0; probe <= set.slot_mask;) {
        uint32_t* slot = set.slots + (size_t)h * kSlotWords;
        // a slot that reads as full is final, and all of it lies in the same cache line
        const uint4 head = *reinterpret_cast<const uint4*>(slot);
        uint32_t st = head.x;
        uint32_t first[3] = {head.y, head.z, head.w};
        const bool plain = (st & kSlotFull) != 0u;
        if (!plain) {
            // empty, locked, or a stale line (a die's L2 keeps a slot as it was when its neighbour was
            // asked for): it is read past the caches, and locked only if it is free (additions to one
            // address are served one after the other)
            const uint64_t* words = reinterpret_cast<const uint64_t*>(slot);
            const uint64_t a = __hip_atomic_load(words, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            st = (uint32_t)a;
            if (st == kSlotEmpty && atomicCAS(slot, kSlotEmpty, kSlotLocked) == kSlotEmpty) {
                // this lane owns the slot: is there still room in T?
                const unsigned long long number = atomicAdd(set.counters, 1ull);
                if ((int64_t)number >= set.cap_T) {
                    atomicOr(set.err, kDevCapacity);
                } else {
                    uint32_t* item = set.members + number * kItemWords;
#pragma unroll
                    for (int k = 0; k < kMaxVecWords; ++k) item[k] = k < NW ? w[k < NW ? k : 0] : 0u;
                    item[kMaxVecWords] = h;
                    set.ranks[number] = 0u;
                }
                slot[kSlotNumber] = (uint32_t)number;
#pragma unroll
                for (int k = 0; k < NW; ++k)
                    __hip_atomic_store(slot + kSlotVector + k, w[k], __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
                // The vector is written past the caches, so "full" may follow as soon as that is done:
                // every word of a slot that others read in this launch has to be stored like that.  (A
                // release here writes back what the die's L2 holds, for every new vector: 97 M rows with
                // 15,609 vectors took 0.79 ms, 0.37 without it.)
                wait_memory();
                __hip_atomic_store(slot, kSlotFull | (uint32_t)number, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
                return (int32_t)number;
            }
            if ((st & kSlotFull) == 0u) {
                // somebody is writing this slot's vector: look again
                if (++spins > set.spin_limit) {
                    atomicOr(set.err, kDevStall);
                    __hip_atomic_store(set.counters + 2, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    return -1;
                }
                __builtin_amdgcn_s_sleep(1);
                continue;
            }
            first[0] = (uint32_t)(a >> 32);
        }
        // The slot is full; only words that came with the state, or are read from here on, decide.  (Words
        // read before it was full are those of the call before: emptying a slot leaves its vector there.)
        wait_memory();
        if (NW > 1 && !plain) {
            const uint64_t b = __hip_atomic_load(reinterpret_cast<const uint64_t*>(slot) + 1, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
            first[1] = (uint32_t)b, first[2] = (uint32_t)(b >> 32);
        }
        auto word_past_caches = [&](int k) {
            return __hip_atomic_load(slot + kSlotVector + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };
        bool same = true;
#pragma unroll
        for (int k = 0; k < NW; ++k)
            same = same && (k < 3 ? first[k < 3 ? k : 0] : plain ? slot[kSlotVector + k] : word_past_caches(k)) == w[k];
        // Another vector, says a line of the caches: what lies behind them decides.  (Hardly a vector meets
        // another one's slot.)
        if (!same && plain) {
            same = true;
#pragma unroll
            for (int k = 0; k < NW; ++k) same = same && word_past_caches(k) == w[k];
        }
        if (same) return (int32_t)(st & ~kSlotFull);
        h = (h + 1u) & set.slot_mask;
        probe += 1;
    }
    return -1;
}

// The LDS tables of a workgroup (kDirectWords + kHashed words, all zero at the start).
//
// Vectors of 2 .. 6 counts have two of them.  The first is a plain array: where the first count is
// zero (every row but the seed's own) and the others are small, the counts themselves, a few bits
// each, are the index, so nothing is hashed and nothing compared, and an entry (number + 1, 0 =
// not known yet) may be written by anybody at any time.  Nearly all rows are of that kind: a node
// that one or a few of a seed's walks met.  The second, for the rest, is a cache of (vector ->
// number) with entries of one LDS read.  (All rows went through a hashed cache before: 25 against
// about 60 instructions a row, and a wave took as long as its slowest lane's walk through the
// global table.)
// Longer vectors have one cache with entries of as many words as they need.
constexpr int kDirectWords = 4096;
// kHashed: words of the hashed cache, a power of two.  (One or two rows in a hundred come here, some
// 400 to 15,000 different vectors; one that finds both its entries taken is a trip to memory every time.)
// kLonely: see find_or_insert_shared.  Pruning 4 M rows of a table of 4,096 vectors that occur equally
// often took 0.56 ms at m = 14 and 0.32 at m = 4 with a turn for every vector of a wave, 0.18 and 0.13
// with 4 lonely ones (of 1,024 vectors 0.43 and 0.22 against 0.17 and 0.12); a walk's own table, 146 M
// rows with some 1,500 vectors, took the same with both.  The fused kernel has its waves at different
// places and little to gain: 99,991 seeds of M = 61, m = 9 take 0.93 ms with a
// turn for every vector, 0.94 with 4 lonely ones (1.27 when every new vector wrote an L2 back).
struct FusedTables {
    static constexpr int kHashed = 4096;  // 16 KB beside the rows of 16 waves
    static constexpr int kLonely = kWave;
};
struct CollectTables {
    static constexpr int kHashed = 4096;  // 16 KB beside their tiles and lists
    static constexpr int kLonely = 4;
};

__device__ __forceinline__ void set_cache_clear(uint32_t* cache, int n_words, int tid, int n_threads) {
    for (int t = tid; t < n_words; t += n_threads) cache[t] = 0u;
}

template <int LT>
struct DirectIndex {
    static_assert(LT >= 2 && LT <= 6, "direct index of 2 .. 6 counts");
    static constexpr int NW = (LT + 1) / 2;
    static constexpr int kBits = LT == 2 ? 12 : LT == 3 ? 6 : LT == 4 ? 4 : LT == 5 ? 3 : 2;
    static_assert(kBits * (LT - 1) <= 12, "the index must stay inside the table");
    // pair[k] holds entry 2k in its lower and entry 2k + 1 in its upper half (zero past the last).
    // Returns whether the vector has an index; *index is below kDirectWords in any case.
    static __device__ __forceinline__ bool of(const uint32_t (&pair)[NW], uint32_t* index) {
        constexpr uint32_t kMost = (1u << kBits) - 1u;
        uint32_t outside = pair[0] & ~(kMost << 16);
        uint32_t at = 0;
#pragma unroll
        for (int k = 1; k < NW; ++k) outside |= pair[k] & ~(kMost << 16 | kMost);
#pragma unroll
        for (int e = 1; e < LT; ++e)
            at |= ((pair[e / 2] >> (e % 2 ? 16 : 0)) & kMost) << (kBits * (e - 1));
        *index = at;
        return outside == 0u;
    }
};

// find_or_insert for the lanes with `pending` set (all lanes of the wavefront call it together).
// One lane goes to the global table for all lanes with the same vector: when a kernel starts,
// nothing is known yet and every row is looked up there, most of them one of a handful of vectors,
// and additions to one address are served one after the other, 13 ns each (350,000 of them, from
// all waves' first tiles, were 3 ms of the pruning of 138 M rows).
// A turn of the loop finds the lanes that share one vector; it ends after Tables::kLonely vectors
// that no other lane shares, for then the rest are mostly such, and every lane left goes for itself.
template <int NW, typename Tables>
__device__ __forceinline__ int32_t find_or_insert_shared(const uint32_t (&w)[NW], uint32_t h,
                                                         bool pending, const VectorSet& set, int lane) {
    int leader = lane;
    bool open = pending;
    int lonely = 0;
    for (uint64_t left = __ballot(open); left != 0ull && lonely < Tables::kLonely; left = __ballot(open)) {
        const int first = __builtin_ctzll(left);
        bool same = open;
#pragma unroll
        for (int k = 0; k < NW; ++k) same = same && wave_bcast_u32(w[k], first) == w[k];
        if constexpr (Tables::kLonely < kWave) lonely += __popcll(__ballot(same)) == 1 ? 1 : 0;
        if (same) leader = first, open = false;
    }
    int32_t number = -1;
    if (pending && leader == lane) number = find_or_insert<NW>(w, h, set);
    return __shfl(number, leader, kWave);
}

// The number of vector w from the hashed cache or the global table (all lanes call it together,
// those without `valid` get -1).  Entries of vectors of at most three words: [0] 0 = free, 1 =
// being written, 2^31 | number = valid; [1 .. NW] the vector; 2 words for NW = 1, else 4, so that
// an entry is one LDS read.  Should the read ever see the valid word next to vector words that are
// not yet there, the comparison fails and the lane asks the global table, which is slower and
// right; a valid entry never changes again.
constexpr uint32_t kPackedValid = 0x80000000u;
template <int NW>
__host__ __device__ constexpr int packed_words() { return NW == 1 ? 2 : 4; }
template <int NW, typename Tables>
__device__ __forceinline__ uint32_t* packed_pair(uint32_t hv, uint32_t* cache) {
    static_assert(NW >= 1 && NW <= 3, "packed cache entries hold up to three words");
    constexpr int EW = packed_words<NW>();
    return cache + ((hv >> 18) & (uint32_t)(Tables::kHashed / EW / 2 - 1)) * (2 * EW);
}

// The number of vector w from the cache alone, -1 if it is not there.
template <int NW, typename Tables>
__device__ __forceinline__ int32_t cached_number(const uint32_t (&w)[NW], uint32_t hv, uint32_t* cache) {
    constexpr int EW = packed_words<NW>();
    const uint32_t* pair = packed_pair<NW, Tables>(hv, cache);
    int32_t number = -1;
#pragma unroll
    for (int place = 0; place < 2; ++place) {
        uint32_t e[4] = {0u, 0u, 0u, 0u};
        if constexpr (EW == 2) {
            const uint2 v = reinterpret_cast<const uint2*>(pair)[place];
            e[0] = v.x, e[1] = v.y;
        } else {
            const uint4 v = reinterpret_cast<const uint4*>(pair)[place];
            e[0] = v.x, e[1] = v.y, e[2] = v.z, e[3] = v.w;
        }
        bool same = (e[0] & kPackedValid) != 0u;
#pragma unroll
        for (int k = 0; k < NW; ++k) same = same && e[1 + k] == w[k];
        number = same ? (int32_t)(e[0] & ~kPackedValid) : number;
    }
    return number;
}

template <int NW, typename Tables>
__device__ __forceinline__ int32_t lookup_hashed(const uint32_t (&w)[NW], uint32_t hv, bool valid,
                                                 uint32_t* cache, const VectorSet& set, int lane) {
    int32_t number = cached_number<NW, Tables>(w, hv, cache);
    const bool miss = valid && number < 0;
    if (__ballot(miss) != 0ull) {
        const int32_t found = find_or_insert_shared<NW, Tables>(w, hv & set.slot_mask, miss, set, lane);
        if (miss) number = found;
        uint32_t* entry = packed_pair<NW, Tables>(hv, cache);
        bool taken = miss && found >= 0;
        if (taken && atomicCAS(entry, 0u, 1u) != 0u) {
            entry += packed_words<NW>();
            taken = atomicCAS(entry, 0u, 1u) == 0u;
        }
        if (taken) {
#pragma unroll
            for (int k = 0; k < NW; ++k) entry[1 + k] = w[k];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __hip_atomic_store(entry, kPackedValid | (uint32_t)found, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
    return valid ? number : -1;
}

// The same for vectors of nw <= kMaxVecWords words (the others zero): entries of 2 + nw words
// (state, number, vector).  An entry is written once, by the lane that wins its state word, and is
// valid for good after that (state, then vector and number, then "valid": LDS operations of a wave
// take effect in order).
template <typename Tables>
__device__ __forceinline__ int32_t lookup_any(const uint32_t (&w)[kMaxVecWords], bool valid, int nw,
                                              uint32_t* cache, const VectorSet& set, int lane) {
    int entries = 64;
    while (entries * 2 * (2 + nw) <= kDirectWords + Tables::kHashed) entries *= 2;
    const uint32_t hv = hash_vector<kMaxVecWords>(w);
    uint32_t* entry = cache + ((hv >> 18) & (uint32_t)(entries - 1)) * (2 + nw);
    bool hit = valid && entry[0] == 2u;
#pragma unroll
    for (int k = 0; k < kMaxVecWords; ++k)
        if (k < nw) hit = hit && entry[2 + k] == w[k];
    const bool miss = valid && !hit;
    int32_t number = hit ? (int32_t)entry[1] : -1;
    if (__ballot(miss) != 0ull) {
        const int32_t found = find_or_insert_shared<kMaxVecWords, Tables>(w, hv & set.slot_mask, miss, set, lane);
        if (miss) number = found;
        if (miss && found >= 0 && atomicCAS(entry, 0u, 1u) == 0u) {
#pragma unroll
            for (int k = 0; k < kMaxVecWords; ++k)
                if (k < nw) entry[2 + k] = w[k];
            entry[1] = (uint32_t)found;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __hip_atomic_store(entry, 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
    return number;
}

// The vector of row t among the rows at cnt16 (LDS, densely packed), as the aligned words that
// cover it, shifted into place: pair[k] holds entry 2k in its lower and 2k + 1 in its upper half.
// n_words: words that hold rows.
template <int NW>
__device__ __forceinline__ void row_pairs(const uint32_t* words, int odd, int n_words, int t, int L,
                                          uint32_t (&pair)[NW]) {
    const int first = odd + t * L;
    const uint32_t shift = (uint32_t)(first & 1) * 2u;
    uint32_t raw[NW + 1];
#pragma unroll
    for (int k = 0; k <= NW; ++k) raw[k] = 2 * k <= L ? words[min((first >> 1) + k, n_words - 1)] : 0u;
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        pair[k] = __builtin_amdgcn_alignbyte(raw[k + 1], raw[k], shift);
        if (2 * k + 1 >= L) pair[k] &= 0xFFFFu;  // the upper half is the next row's
        if (2 * k >= L) pair[k] = 0u;
    }
}

// Looks the rows misses[0 .. n_miss) of the rows at cnt16 up (words, odd, n_words as for row_pairs)
// and enters what belongs there into the direct table.
template <int LT, typename Tables>
__device__ __forceinline__ void resolve_misses(const uint16_t* misses, int n_miss, int lane,
                                               const uint32_t* words, int odd, int n_words,
                                               uint32_t* cache, const VectorSet& set,
                                               int32_t* __restrict__ code) {
    constexpr int NW = (LT + 1) / 2;
    for (int u0 = 0; u0 < n_miss; u0 += kWave) {
        const bool valid = u0 + lane < n_miss;
        const int t = (int)misses[valid ? u0 + lane : 0];
        uint32_t pair[NW], w[NW], at;
        row_pairs<NW>(words, odd, n_words, t, LT, pair);
        const bool small = DirectIndex<LT>::of(pair, &at);
#pragma unroll
        for (int k = 0; k < NW; ++k) w[k] = (pair[k] << 16) | (pair[k] >> 16);
        const int32_t number =
            lookup_hashed<NW, Tables>(w, hash_vector<NW>(w), valid, cache + kDirectWords, set, lane);
        if (valid && small && number >= 0) cache[at] = (uint32_t)number + 1u;
        if (valid) code[t] = number;
    }
}

// The lanes with `miss` set append their row t to the list.
__device__ __forceinline__ void append_misses(uint16_t* misses, int& n_miss, bool miss, int t) {
    const uint64_t all = __ballot(miss);
    if (all == 0ull) return;
    const int before = (int)__builtin_amdgcn_mbcnt_hi(
        (uint32_t)(all >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)all, 0u));
    if (miss) misses[n_miss + before] = (uint16_t)t;
    n_miss += __popcll(all);
}

// The numbers of n rows whose counts lie in LDS, to code[0 .. n).  One wavefront; rows that are not
// in the direct table are put on a list (misses, n places in LDS of the wave's own) and looked up
// together afterwards, so that few lanes wait for few.  LT = m + 1 at compile time for 2 .. 6, 0 =
// any.
template <int LT, typename Tables>
__device__ __forceinline__ void rows_numbers(int n, int lane, int L, const uint16_t* cnt16,
                                             uint16_t* misses, uint32_t* cache, const VectorSet& set,
                                             int32_t* __restrict__ code) {
    const int odd = (int)((reinterpret_cast<uintptr_t>(cnt16) >> 1) & 1u);
    const uint32_t* words = reinterpret_cast<const uint32_t*>(cnt16 - odd);
    const int n_words = (odd + n * L + 1) / 2;
    if constexpr (LT == 0) {
        for (int t0 = 0; t0 < n; t0 += kWave) {
            const int t = t0 + lane;
            uint32_t pair[kMaxVecWords], w[kMaxVecWords];
            row_pairs<kMaxVecWords>(words, odd, n_words, min(t, n - 1), L, pair);
#pragma unroll
            for (int k = 0; k < kMaxVecWords; ++k) w[k] = (pair[k] << 16) | (pair[k] >> 16);
            const int32_t number = lookup_any<Tables>(w, t < n, (L + 1) / 2, cache, set, lane);
            if (t < n) code[t] = number;
        }
    } else {
        constexpr int NW = (LT + 1) / 2;
        int n_miss = 0;
        for (int t0 = 0; t0 < n; t0 += kWave) {
            const int t = t0 + lane;
            uint32_t pair[NW], at;
            row_pairs<NW>(words, odd, n_words, min(t, n - 1), LT, pair);
            const bool small = DirectIndex<LT>::of(pair, &at);
            const uint32_t e = cache[at];
            const bool hit = small && e != 0u;
            if (t < n && hit) code[t] = (int32_t)(e - 1u);
            append_misses(misses, n_miss, t < n && !hit, t);
        }
        wave_sync();
        resolve_misses<LT, Tables>(misses, n_miss, lane, words, odd, n_words, cache, set, code);
        wave_sync();
    }
}
template <typename Tables>
__device__ __forceinline__ void rows_numbers_any(int n, int lane, int L, const uint16_t* cnt16,
                                                 uint16_t* misses, uint32_t* cache,
                                                 const VectorSet& set, int32_t* __restrict__ code) {
    switch (L) {
        case 2: rows_numbers<2, Tables>(n, lane, L, cnt16, misses, cache, set, code); break;
        case 3: rows_numbers<3, Tables>(n, lane, L, cnt16, misses, cache, set, code); break;
        case 4: rows_numbers<4, Tables>(n, lane, L, cnt16, misses, cache, set, code); break;
        case 5: rows_numbers<5, Tables>(n, lane, L, cnt16, misses, cache, set, code); break;
        case 6: rows_numbers<6, Tables>(n, lane, L, cnt16, misses, cache, set, code); break;
        default: rows_numbers<0, Tables>(n, lane, L, cnt16, misses, cache, set, code); break;
    }
}

}  // namespace surel
