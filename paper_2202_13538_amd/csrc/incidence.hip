// The queries of every node (Sec. 3.6 "Mini-batching for Training": two nodes are neighbours
// when a query holds both, so the search walks node -> its queries -> their nodes).  Built by a
// stable radix sort of the (node, query) pairs of the query list: inc_q holds, node by node,
// the indices of the queries that name the node, ascending; inc_off[x] .. inc_off[x+1] is
// node x's part.
//
// One pass puts the pairs into buckets of consecutive nodes (the node's upper bits, at most 1,024
// buckets), in three launches: digit counts of every tile, places (column sums over the tiles and
// over the digits), and the scatter, which puts a tile's pairs in order in LDS first, so that they
// leave as runs of a bucket.  Then a workgroup per bucket sorts its pairs by the node's lower bits in
// LDS, and writes the nodes' offsets and the queries: they go through memory once.  Buckets with more
// pairs than LDS holds (queries crowd on neighbouring nodes) are cut into chunks; the same launch counts
// each chunk's nodes, and another one puts the chunks in order.
// What bounds it: the memory round trips of the launches one after the other, at these sizes: a million
// two-node queries on 2.9M nodes 39 us (4.7 + 5.9 + 12.6 + 15 + 3.8 in a trace, of which the last finds that there
// are no chunks), with three passes of 8 bits and the offsets behind them 85.
// Graphs of up to 255 nodes, for which one pass of 8 bits does, and graphs of 2^23 nodes and more, whose
// buckets would have more nodes than LDS has room for, are sorted 8 bits a pass, least significant first, the
// same three launches a pass, and the offsets by a launch of their own.
#include "device_util.h"
#include "kernels.h"
#include "small_scan.h"

namespace surel {

namespace {

constexpr int kSortThreads = 1024;
constexpr int kSortWaves = kSortThreads / kWave;
constexpr int kSortBins = 256;                    // 8 bits a pass
constexpr int kBucketBits = 10;                   // at most 2^10 buckets
constexpr int kBuckets = 1 << kBucketBits;
constexpr int kSortMostItems = 8;                 // pairs per thread of a tile
constexpr int kSortFewItems = 2;                  // for short lists: more tiles than compute units
constexpr int64_t kSortFew = 1 << 19;

// Where a pass takes its pairs from: the query list (entry t names node queries[t] and belongs to
// query t / k; an id outside the graph sorts behind every node's part) or the pass before.
struct SortSource {
    const int32_t* queries;  // or null
    int32_t k;
    int32_t n_nodes;
    const uint2* pairs;
    uint32_t* err;
    __device__ __forceinline__ uint2 get(int64_t t, bool* bad) const {
        if (queries == nullptr) return pairs[t];
        const uint32_t x = (uint32_t)queries[t];
        const bool out = x >= (uint32_t)n_nodes;
        *bad = *bad || out;
        const uint32_t at = (uint32_t)t;  // t / k for k = 1, 2, 3
        const uint32_t query = k == 1 ? at : k == 2 ? at >> 1 : __umulhi(at, 0xAAAAAAABu) >> 1;
        return make_uint2(out ? (uint32_t)n_nodes : x, query);
    }
};

// Where the scatter puts a pair: whole, or (last pass) apart, or as an item of a bucket, the lower
// bits of the node above the query's number, in as few bytes as hold both.
struct SortTarget {
    uint2* pairs;
    uint32_t* keys;
    int32_t* vals;
    void* items;
    int low_bits, query_bits;
    __device__ __forceinline__ void put(uint32_t to, uint2 p) const {
        if (items != nullptr) {
            const uint32_t low = p.x & ((1u << low_bits) - 1u);
            if (low_bits + query_bits <= 32) {
                static_cast<uint32_t*>(items)[to] = low << query_bits | p.y;
            } else {
                static_cast<uint64_t*>(items)[to] = (uint64_t)low << query_bits | p.y;
            }
        } else if (keys == nullptr) {
            pairs[to] = p;
        } else {
            keys[to] = p.x;
            vals[to] = (int32_t)p.y;
        }
    }
};

// hist[tile][d] = pairs of the tile whose key has digit d.
template <int kItems, int kBins>
__global__ __launch_bounds__(kSortThreads) void sort_hist_kernel(SortSource src, int64_t n, int shift,
                                                                uint32_t* __restrict__ hist,
                                                                uint32_t* __restrict__ any_large) {
    __shared__ uint32_t bins[kBins];
    const int tid = (int)threadIdx.x;
    if (any_large != nullptr && blockIdx.x == 0 && tid == 0) *any_large = 0u;
    if (tid < kBins) bins[tid] = 0u;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kSortThreads * kItems;
    uint2 pair[kItems];
    bool bad = false;
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const int64_t t = base + r * kSortThreads + tid;
        pair[r] = t < n ? src.get(t, &bad) : make_uint2(0u, 0u);
    }
#pragma unroll
    for (int r = 0; r < kItems; ++r)
        if (base + r * kSortThreads + tid < n)
            atomicAdd(&bins[(pair[r].x >> shift) & (kBins - 1)], 1u);
    __syncthreads();
    if (tid < kBins) hist[(int64_t)blockIdx.x * kBins + tid] = bins[tid];
    raise_error(src.err, bad, kDevBadQuery);
}

// places[tile][d] = place of the tile's first pair with digit d.  A workgroup takes 64 digits, its
// 16 waves a share of the tiles each; the digits of the workgroups before it come in through
// small_scan.h (whose helpers read the counts at any time: the places are an array of their own).
// any_large (optional; the counting launch has cleared it): set where a digit has more than `large` pairs.
template <int kBins>
__global__ __launch_bounds__(kSortThreads) void sort_places_kernel(const uint32_t* __restrict__ hist,
                                                                  int64_t n_tiles,
                                                                  uint32_t* __restrict__ places,
                                                                  SmallScan* __restrict__ ss,
                                                                  uint32_t spin_limit, uint32_t large,
                                                                  uint32_t* __restrict__ any_large) {
    __shared__ uint32_t share[kSortWaves][kWave];
    __shared__ int64_t s_base;
    const int lane = lane_id();
    const int wave = (int)(threadIdx.x >> 6);
    const int64_t per_wave = (n_tiles + kSortWaves - 1) / kSortWaves;
    const int64_t t0 = wave * per_wave, t1 = min(t0 + per_wave, n_tiles);
    const uint32_t* column = hist + (int64_t)blockIdx.x * kWave + lane;
    uint32_t* to = places + (int64_t)blockIdx.x * kWave + lane;
    uint32_t tag = 0;
    if (wave == 0) tag = small_scan_tag(ss);
    constexpr int kPlaceTiles = kBins == kBuckets ? 16 : 8;
    uint32_t first[kPlaceTiles], sum = 0;  // the wave's first tiles stay in registers
#pragma unroll
    for (int u = 0; u < kPlaceTiles; ++u) first[u] = t0 + u < t1 ? column[(t0 + u) * kBins] : 0u;
#pragma unroll
    for (int u = 0; u < kPlaceTiles; ++u) sum += first[u];
    for (int64_t t = t0 + kPlaceTiles; t < t1; t += 4) {
        uint32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = t + u < t1 ? column[(t + u) * kBins] : 0u;
#pragma unroll
        for (int u = 0; u < 4; ++u) sum += v[u];
    }
    share[wave][lane] = sum;
    __syncthreads();
    uint32_t before = 0, total = 0;  // of this digit: pairs of the waves before, of all waves
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) {
        if (w < wave) before += share[w][lane];
        total += share[w][lane];
    }
    const uint32_t incl = wave_incl_sum(total);
    if (wave == 0) {
        if (any_large != nullptr && total > large) *any_large = 1u;
        if (lane == kWave - 1) small_scan_publish(ss, (int)blockIdx.x, tag, incl);
        const int64_t base =
            small_scan_before(ss, (int)blockIdx.x, tag, spin_limit, lane, [&](int j) {
                uint32_t pairs = 0;  // of another workgroup's digits
#pragma unroll 1
                for (int64_t t = 0; t < n_tiles; ++t) pairs += hist[t * kBins + j * kWave + lane];
                return wave_bcast_u32(wave_incl_sum(pairs), kWave - 1);
            });
        if (lane == 0) {
            small_scan_done(ss, (int)blockIdx.x, tag, (int)gridDim.x);
            s_base = base;
        }
    }
    __syncthreads();
    uint32_t at = (uint32_t)s_base + incl - total + before;
#pragma unroll
    for (int u = 0; u < kPlaceTiles; ++u) {
        if (t0 + u < t1) to[(t0 + u) * kBins] = at;
        at += first[u];
    }
    for (int64_t t = t0 + kPlaceTiles; t < t1; t += 4) {
        uint32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = t + u < t1 ? column[(t + u) * kBins] : 0u;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (t + u < t1) to[(t + u) * kBins] = at;
            at += v[u];
        }
    }
}

// Moves a tile's pairs to their places.  Wave w owns the tile's pairs [w * 64 * kItems, ..) in
// rounds of 64, in index order: a pair's rank among the earlier ones of its digit is that of its
// wave so far, plus the lanes before it with the same digit.
// kFast: one addition in LDS that returns the count before it gives both, if it takes the lanes one after
// the other (as LDS does).  Whether it did shows in the sorted tile, whose pairs' queries ascend inside a
// digit; else, and where pairs come in another order than that of the queries, ballots tell, one a bit.
// 2.1 M pairs to 708 buckets 12.3 us, with ballots 15.
template <int kItems, int kBins, bool kFast>
__global__ __launch_bounds__(kSortThreads) void sort_scatter_kernel(
    SortSource src, int64_t n, int shift, const uint32_t* __restrict__ places, SortTarget target) {
    // pairs of a digit in a wave, then before it: 16 bits each
    __shared__ __align__(16) uint32_t count_words[kSortWaves][kBins / 2];
    __shared__ uint32_t start[kBins];              // first place of a digit inside the tile
    __shared__ uint32_t shift_to[kBins];           // its place in the output minus that
    __shared__ uint32_t wave_sum[kBins / kWave];
    extern __shared__ __align__(16) uint2 sorted[];    // the tile's pairs, in order
    const int tid = (int)threadIdx.x;
    const int lane = lane_id();
    const int wave = tid >> 6;
    uint16_t* count = reinterpret_cast<uint16_t*>(&count_words[0][0]);  // [wave][digit]
    uint16_t* own = count + wave * kBins;
    const int64_t tile = (int64_t)blockIdx.x * kSortThreads * kItems;
    const int64_t base = tile + wave * (kWave * kItems);
    uint2 pair[kItems];
    bool bad = false;
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const int64_t t = base + r * kWave + lane;
        pair[r] = t < n ? src.get(t, &bad) : make_uint2(0u, 0u);
    }
    const uint64_t below = (1ull << lane) - 1ull;
    const int n_here = (int)min((int64_t)kSortThreads * kItems, n - tile);
#pragma unroll 1
    for (bool fast = kFast;; fast = false) {
        for (int d = lane; d < kBins / 8; d += kWave)
            reinterpret_cast<uint4*>(own)[d] = make_uint4(0u, 0u, 0u, 0u);
        wave_sync();
        uint32_t rank[kItems];
        if (fast) {
#pragma unroll
            for (int r = 0; r < kItems; ++r) {
                const uint32_t d = (pair[r].x >> shift) & (kBins - 1);
                if (base + r * kWave + lane < n)
                    rank[r] = atomicAdd(&count_words[wave][d >> 1], 1u << (d & 1u) * 16u) >> (d & 1u) * 16u & 0xFFFFu;
            }
        } else {
#pragma unroll
            for (int r = 0; r < kItems; ++r) {
                const bool valid = base + r * kWave + lane < n;
                uint32_t d = (pair[r].x >> shift) & (kBins - 1);
                if (kFast) asm volatile("" : "+v"(d));  // (its bits are not looked at before they are needed)
                uint64_t same = __ballot(valid);  // lanes whose pair has this lane's digit
#pragma unroll
                for (int b = 0; (1 << b) < kBins; ++b) {
                    const uint64_t has = __ballot((d >> b) & 1u);
                    same &= ((d >> b) & 1u) ? has : ~has;
                }
                const uint32_t in_round = (uint32_t)__popcll(same & below);
                const uint32_t group = (uint32_t)__popcll(same);
                const uint32_t so_far = own[d];
                rank[r] = so_far + in_round;
                wave_sync();  // every lane has read the count before the group's last lane moves it on
                if (valid && in_round + 1 == group) own[d] = (uint16_t)(so_far + group);
                wave_sync();
            }
        }
        __syncthreads();
        uint32_t total = 0;
        if (tid < kBins) {
#pragma unroll
            for (int w = 0; w < kSortWaves; ++w) {
                const uint32_t c = count[w * kBins + tid];
                count[w * kBins + tid] = (uint16_t)total;
                total += c;
            }
        }
        uint32_t incl = 0;
        if (wave < kBins / kWave) {
            incl = wave_incl_sum(total);
            if (lane == kWave - 1) wave_sum[wave] = incl;
        }
        __syncthreads();
        if (tid < kBins) {
            uint32_t first = incl - total;
            for (int w = 0; w < wave; ++w) first += wave_sum[w];
            start[tid] = first;
            shift_to[tid] = places[(int64_t)blockIdx.x * kBins + tid] - first;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kItems; ++r) {
            if (base + r * kWave + lane < n) {
                const uint32_t d = (pair[r].x >> shift) & (kBins - 1);
                sorted[start[d] + own[d] + rank[r]] = pair[r];
            }
        }
        __syncthreads();
        bool wrong = false;
#pragma unroll
        for (int r = 0; r < kItems; ++r) {
            const int i = r * kSortThreads + tid;
            if (i < n_here) {
                const uint2 p = sorted[i];
                const uint32_t d = (p.x >> shift) & (kBins - 1);
                if (fast) {
                    const uint2 next = sorted[min(i + 1, n_here - 1)];
                    wrong = wrong || (next.y < p.y && ((next.x >> shift) & (kBins - 1)) == d);
                }
                const uint32_t to = shift_to[d] + (uint32_t)i;
                // (a place is one of the output unless the list changes while it is sorted)
                if (to < (uint32_t)n) target.put(to, p);
            }
        }
        if (!fast || __syncthreads_or(wrong) == 0) break;
    }
}

// First index in [0, n) whose key is not below value (n if none): one wavefront, 64 pivots a step.
__device__ __forceinline__ int64_t wave_lower_bound(const uint32_t* __restrict__ keys, int64_t n,
                                                    int64_t value, int lane) {
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t step = (hi - lo + kWave - 1) / kWave;
        const int64_t p = lo + (lane + 1) * step - 1;  // the last key of the lane's part
        const bool below = p < hi && (int64_t)keys[min(p, n - 1)] < value;
        const int64_t parts = __popcll(__ballot(below));
        const int64_t next = lo + parts * step;  // one past the last pivot below value: hi at most
        hi = min(hi, next + step - 1);
        lo = next;
    }
    return lo;
}

// inc_off[x] = number of sorted keys below x, for x = 0..n_nodes.  A workgroup's nodes are
// consecutive: two waves find where their keys begin and end, the place behind a node's last key is
// noted in LDS, and a node's offset is the largest such place of the nodes before it.
// What bounds it: the chain of a workgroup (four trips of the search, the keys, the scan), so all
// workgroups are to be on the device at once: 512 of them, up to the nodes whose places LDS holds.
// 2.9M nodes and 2.1M keys: 11.7 us; with 1,024 nodes to a workgroup of four waves, each searched
// for in the LDS copy of the keys, 22.
// Where a workgroup has more keys than kOffsetsKeys (a few nodes hold most of the list), its nodes
// are searched for in the list itself, which takes no longer for a longer list.
constexpr int kOffsetsThreads = 1024;
constexpr int kOffsetsItems = 8;      // nodes of a thread, at most
constexpr int kOffsetsGroups = 512;   // two workgroups per compute unit
constexpr int64_t kOffsetsKeys = 1 << 16;
int offsets_items(int32_t n_nodes) {
    const int64_t want = ((int64_t)n_nodes + 1 + kOffsetsThreads * kOffsetsGroups - 1) /
                         (kOffsetsThreads * kOffsetsGroups);
    return want < kOffsetsItems ? (int)want : kOffsetsItems;
}
__global__ __launch_bounds__(kOffsetsThreads) void incidence_offsets_kernel(
    const uint32_t* __restrict__ keys, int64_t n, int32_t n_nodes, int items,
    int64_t* __restrict__ inc_off) {
    __shared__ int32_t behind[kOffsetsThreads * kOffsetsItems];  // place behind the node's last key
    __shared__ int32_t wave_most[kOffsetsThreads / kWave];
    __shared__ int64_t ends[2];
    const int tid = (int)threadIdx.x;
    const int lane = lane_id();
    const int wave = tid >> 6;
    const int n_here = kOffsetsThreads * items;
    const int64_t x0 = (int64_t)blockIdx.x * n_here;
    if (wave < 2) {
        const int64_t at = wave_lower_bound(keys, n, x0 + wave * n_here, lane);
        if (lane == 0) ends[wave] = at;
    }
    for (int t = tid; t < n_here; t += kOffsetsThreads) behind[t] = 0;
    __syncthreads();
    const int64_t first = ends[0], n_near = ends[1] - first;
    if (n_near > kOffsetsKeys) {
        for (int64_t x = x0 + tid; x < x0 + n_here && x <= n_nodes; x += kOffsetsThreads) {
            int64_t lo = first, hi = ends[1];
            while (lo < hi) {
                const int64_t mid = (lo + hi) >> 1;
                if ((int64_t)keys[mid] < x) {
                    lo = mid + 1;
                } else {
                    hi = mid;
                }
            }
            inc_off[x] = lo;
        }
        return;
    }
    const uint32_t* near_keys = keys + first;
    constexpr int kFlight = 4;  // keys a thread has in flight
    for (int t0 = 0; t0 < (int)n_near; t0 += kFlight * kOffsetsThreads) {
        uint32_t key[kFlight], next[kFlight];
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
            const int t = t0 + u * kOffsetsThreads + tid;
            key[u] = near_keys[min(t, (int)n_near - 1)];
            next[u] = near_keys[min(t + 1, (int)n_near - 1)];
        }
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
            const int t = t0 + u * kOffsetsThreads + tid;
            // (a key is one of the workgroup's nodes unless the list changes while it is sorted)
            const uint32_t at = key[u] - (uint32_t)x0;
            if (t < (int)n_near && at < (uint32_t)n_here && (key[u] != next[u] || t + 1 == (int)n_near))
                behind[at] = t + 1;
        }
    }
    __syncthreads();
    // the largest of the nodes before: of the thread's own, of the lanes before, of the waves before
    int32_t most = 0;
    for (int u = 0; u < items; ++u) most = max(most, behind[tid * items + u]);
    int32_t incl = most;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int32_t other = __shfl_up(incl, d, kWave);
        if (lane >= d) incl = max(incl, other);
    }
    if (lane == kWave - 1) wave_most[wave] = incl;
    const int32_t below = __shfl_up(incl, 1, kWave);
    __syncthreads();
    int32_t before = lane > 0 ? below : 0;
    for (int w = 0; w < wave; ++w) before = max(before, wave_most[w]);
    for (int u = 0; u < items; ++u) {
        const int32_t own = behind[tid * items + u];
        behind[tid * items + u] = before;
        before = max(before, own);
    }
    __syncthreads();
    for (int t = tid; t < n_here; t += kOffsetsThreads)
        if (x0 + t <= n_nodes) inc_off[x0 + t] = first + behind[t];
}

// The buckets' lists.  A workgroup takes the pairs of its bucket in order, a share of consecutive ones a
// wave: they are counted for every wave and node, sums over both give each node's place and, within it,
// each wave's, and counting once more puts the pairs there.
// What bounds it: a third each the way there (launch, the bucket's place, its pairs), instructions, and
// 8 bytes a node and 4 a pair on their way out.  708 buckets of 3,000 pairs and 4,096 nodes 14 us; with
// pairs read twice and the offsets last 18.5, sorted in two passes of six bits 27.
//
// Lists that crowd.  Where a byte does not count a node's pairs of a wave, and in the chunks of large buckets,
// ballots tell a round's pairs of a node apart, and the waves take turns to add theirs to the nodes' words.
// What bounds the chunks is that every one reads the counts of all chunks of its bucket: 2.1 M pairs on 3,000
// neighbours of 2.9M nodes, 205 chunks of 4,096 counts, 55 us, 26 of them the counts (16 the turns, 5 the way
// out through LDS, 24 without it).  The whole call in us, 8 bits a pass / chunks of 6,656 pairs sorted in two
// passes by 256 threads of the launch for the buckets / as it is, 2.1 M pairs on 2.9M nodes and on 235,000:
//    half of them with one node      122 / 127 /  84     99 / 110 /  60
//    all with one node               117 / 155 / 102     97 / 125 /  71
//    3,000 neighbours                132 / 160 / 107     98 / 105 /  60
//    1,048 nodes, 2,000 times each    96 / 100 /  83     92 /  95 /  71
//    ids by descending degree        133 / 106 /  73     96 / 103 /  55
constexpr int kListThreads = 256;
constexpr int kListWaves = kListThreads / kWave;
static_assert(kListWaves == 4, "a node's four counts are the bytes of four words");
constexpr int kListRounds = 26;                // pairs of a thread, at most
// of a bucket that LDS takes: with 32-bit items and up to 12 lower bits, of three workgroups a CU
constexpr int kListPairs = kListRounds * kListThreads;
constexpr int kListBits = 13;                  // lower bits of a node, at most
constexpr int kListFlight = 8;    // rows of chunk counts in flight, and a wave's rounds of pairs
constexpr int kListChunks = 256;  // workgroups that count chunks' nodes, and that put chunks in order
constexpr int kChunkThreads = 1024;
constexpr int kChunkWaves = kChunkThreads / kWave;
constexpr int kPartRounds = 10;
constexpr int kPartPairs = kPartRounds * kChunkThreads;  // of a chunk that LDS takes at a time

// Nodes of a bucket, rounded up to whole 16-byte pieces of their counts.
__host__ __device__ constexpr int list_nodes(int low_bits) { return low_bits < 4 ? 16 : 1 << low_bits; }

struct ListJob {
    const uint32_t* any_large;     // not zero: a bucket has more than kListPairs pairs
    const uint32_t* bucket_start;  // of every bucket, in items
    int n_buckets;
    int64_t n;
    const void* items;
    int low_bits, query_bits;
    int32_t n_nodes;
    uint32_t chunk_pairs;          // of a bucket with more than kListPairs
    uint16_t* chunk_counts;        // [chunk][list_nodes(low_bits)]
    int64_t* inc_off;
    int32_t* inc_q;
    // (inside the array also where the query list changes while it is sorted)
    __device__ __forceinline__ uint32_t start_of(int b) const {
        return min(b < n_buckets ? bucket_start[b] : (uint32_t)n, (uint32_t)n);
    }
    template <typename Item>
    __device__ __forceinline__ uint32_t low_of(Item item) const {
        return (uint32_t)(item >> query_bits) & ((1u << low_bits) - 1u);
    }
    __device__ __forceinline__ uint32_t size_of(int b) const {
        const uint32_t first = start_of(b), end = start_of(b + 1);
        return end > first ? end - first : 0u;
    }
};

// Chunk number `id` of the large buckets; bucket -1: there are no more.
struct ListChunk {
    int bucket;
    uint32_t first, n;             // pairs of the chunk, as places among the items
    int at, bucket_chunk, n_bucket_chunks;  // its row of chunk_counts, its bucket's first row, and rows
};
template <int kThreads>
__device__ __forceinline__ ListChunk list_chunk(const ListJob& job, int id, ListChunk* shared,
                                                uint32_t* wave_sum) {
    const int tid = (int)threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    if (*job.any_large == 0u) return ListChunk{-1, 0, 0, 0, 0, 0};
    constexpr int kPer = kBuckets / kThreads;
    uint32_t chunks[kPer], sum = 0;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int b = tid * kPer + u;
        const uint32_t size = b < job.n_buckets ? job.size_of(b) : 0u;
        chunks[u] = size > (uint32_t)kListPairs ? (size + job.chunk_pairs - 1) / job.chunk_pairs : 0u;
        sum += chunks[u];
    }
    __syncthreads();
    if (tid == 0) shared->bucket = -1;
    const uint32_t incl = wave_incl_sum(sum);
    if (lane == kWave - 1) wave_sum[wave] = incl;
    __syncthreads();
    uint32_t first = incl - sum;
    for (int w = 0; w < wave; ++w) first += wave_sum[w];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        if ((uint32_t)id >= first && (uint32_t)id < first + chunks[u]) {
            const int b = tid * kPer + u;
            const uint32_t before = ((uint32_t)id - first) * job.chunk_pairs;
            *shared = ListChunk{b, job.start_of(b) + before, min(job.size_of(b) - before, job.chunk_pairs),
                                id, (int)first, (int)chunks[u]};
        }
        first += chunks[u];
    }
    __syncthreads();
    return *shared;
}

// Pairs of every node of the chunks of large buckets, workgroup `group` of n_groups.  counts: a word a node.
template <typename Item>
__device__ __forceinline__ void list_chunk_counts(const ListJob& job, int group, int n_groups, uint32_t* counts,
                                                  ListChunk* shared, uint32_t* wave_sum) {
    const int tid = (int)threadIdx.x, lane = tid & (kWave - 1);
    const Item* items = static_cast<const Item*>(job.items);
#pragma unroll 1
    for (int id = group;; id += n_groups) {
        const ListChunk c = list_chunk<kListThreads>(job, id, shared, wave_sum);
        if (c.bucket < 0) return;
        for (int x = tid; x < list_nodes(job.low_bits); x += kListThreads) counts[x] = 0u;
        __syncthreads();
        for (uint32_t t0 = 0; t0 < c.n; t0 += 8 * kListThreads) {
            uint32_t low[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const uint32_t t = t0 + u * kListThreads + tid;
                low[u] = job.low_of(items[c.first + min(t, c.n - 1)]);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const bool valid = t0 + u * kListThreads + tid < c.n;
                // a node that holds most of a bucket: one addition for a wave of its pairs
                const uint32_t one = wave_bcast_u32(low[u], 0);
                const uint64_t all = __ballot(valid);
                if (__ballot(valid && low[u] == one) == all) {
                    if (lane == 0 && all != 0ull) atomicAdd(&counts[one], (uint32_t)__popcll(all));
                } else if (valid) {
                    atomicAdd(&counts[low[u]], 1u);
                }
            }
        }
        __syncthreads();
        uint16_t* to = job.chunk_counts + (int64_t)c.at * list_nodes(job.low_bits);
        for (int x = tid; x < list_nodes(job.low_bits); x += kListThreads) to[x] = (uint16_t)counts[x];
        __syncthreads();
    }
}

// What a lane does with its pair in a round of 64, in a word: a place among the nodes' words and what it adds
// there (the first lane of a node the number of its pairs, the others nothing, somewhere), the lane's rank
// among the lanes of its node, and the first of them.
constexpr int kRankAt = kListBits, kLeaderAt = kRankAt + 6, kAddAt = kLeaderAt + 6;
static_assert(kAddAt + 7 <= 32, "a word");

// Rounds of 64 pairs of a wave that has some, of n in all: no fewer than four, for a wave's turn (list_turns)
// takes longer than its rounds.
template <int kThreads>
__device__ __forceinline__ int list_rounds(int n) { return max((n + kThreads - 1) / kThreads, 4); }

// word[r] of round r of the wave's pairs, a share of consecutive ones of n, found by ballots, one a bit.
// totals (or null): a word a node, to which the node's pairs are added.
template <typename Item, int kThreads, int kRounds>
__device__ __forceinline__ void list_ranks(const ListJob& job, const Item* __restrict__ items, int n,
                                           uint32_t (&word)[kRounds], uint32_t* totals) {
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int rounds = list_rounds<kThreads>(n);
    int base = wave * rounds * kWave + lane;
    asm volatile("" : "+v"(base));  // (no comparison is kept from one loop for the next)
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int r0 = 0; r0 < kRounds; r0 += kListFlight) {
        uint32_t low[kListFlight];
        uint64_t same[kListFlight];
        if (r0 < rounds) {
#pragma unroll
            for (int u = 0; u < kListFlight && r0 + u < kRounds; ++u) {
                low[u] = job.low_of(items[min(base + (r0 + u) * kWave, n - 1)]);
                same[u] = __ballot(r0 + u < rounds && base + (r0 + u) * kWave < n);
            }
#pragma unroll 1
            for (int b = 0; b < job.low_bits; ++b) {
#pragma unroll
                for (int u = 0; u < kListFlight && r0 + u < kRounds; ++u) {
                    const bool one = (low[u] >> b & 1u) != 0u;
                    const uint64_t has = __ballot(one);
                    same[u] &= one ? has : ~has;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kListFlight && r0 + u < kRounds; ++u) {
            word[r0 + u] = (uint32_t)lane & 15u;
            if (r0 + u < rounds && base + (r0 + u) * kWave < n) {
                const uint32_t rank = (uint32_t)__popcll(same[u] & below), all = (uint32_t)__popcll(same[u]);
                const uint32_t leader = (uint32_t)__ffsll((unsigned long long)same[u]) - 1u;
                const uint32_t adds = rank == 0u ? low[u] | all << kAddAt : (uint32_t)lane & 15u;
                word[r0 + u] = adds | rank << kRankAt | leader << kLeaderAt;
                if (totals != nullptr && rank == 0u) atomicAdd(&totals[low[u]], all);
            }
        }
    }
}

// place[r] of the pairs of list_ranks, in order of their nodes and queries: words[x] is the place of node x's
// first one and becomes the one behind its last.  The waves take turns, so that a wave's pairs come behind
// those of the waves before; a turn's additions follow one another in LDS, which takes a wave's instructions
// in order.
template <int kThreads, int kRounds>
__device__ __forceinline__ void list_turns(int n, const uint32_t (&word)[kRounds], uint32_t* words,
                                           uint32_t (&place)[kRounds]) {
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int rounds = list_rounds<kThreads>(n);
#pragma unroll
    for (int r = 0; r < kRounds; ++r) place[r] = 0u;
    __syncthreads();
#pragma unroll 1
    for (int turn = 0; turn * rounds * kWave < n; ++turn) {
        if (wave == turn) {
#pragma unroll
            for (int r0 = 0; r0 < kRounds; r0 += kListFlight) {
                if (r0 < rounds) {
#pragma unroll
                    for (int r = r0; r < r0 + kListFlight && r < kRounds; ++r)
                        place[r] = atomicAdd(&words[word[r] & ((1u << kListBits) - 1u)], word[r] >> kAddAt);
                }
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
        place[r] = (word[r] >> kRankAt & 63u) +
                   (uint32_t)__shfl((int)place[r], (int)(word[r] >> kLeaderAt & 63u), kWave);
}

// words[x], pairs of node x, becomes the place of its first one, `first` being that of the bucket's.
// each(x, place): called for every node, before its word changes.
template <int kThreads, typename Each>
__device__ __forceinline__ void list_node_places(int n_here, uint32_t first, uint32_t* words, uint32_t* wave_word,
                                                 Each&& each) {
    const int tid = (int)threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const int turns = (n_here + kThreads - 1) / kThreads;
    __syncthreads();
    uint32_t sum = 0;
#pragma unroll 1
    for (int u = 0; u < turns; ++u) {
        const int x = (wave * turns + u) * kWave + lane;
        sum += x < n_here ? words[x] : 0u;
    }
    sum = wave_bcast_u32(wave_incl_sum(sum), kWave - 1);
    if (lane == 0) wave_word[wave] = sum;
    __syncthreads();
    uint32_t before = first;
    for (int w = 0; w < wave; ++w) before += wave_word[w];
#pragma unroll 1
    for (int u = 0; u < turns; ++u) {
        const int x = (wave * turns + u) * kWave + lane;
        const uint32_t here = x < n_here ? words[x] : 0u;
        const uint32_t incl = wave_incl_sum(here);
        const uint32_t place = before + incl - here;
        if (x < n_here) {
            each(x, place);
            words[x] = place;
        }
        before += wave_bcast_u32(incl, kWave - 1);
    }
    __syncthreads();
}

// LDS of a workgroup: the pairs, then for every node of the bucket its place, and a word.
template <typename Item>
size_t list_lds_bytes(int low_bits) {
    return kListPairs * sizeof(Item) + (size_t)list_nodes(low_bits) * 6;
}

// A bucket's pairs.  counts: a byte for every wave (list_nodes / 4 words apart) and node, cleared; places: 16
// bits for every node.  Where a node has more pairs than a byte holds, or the pairs have not come out in
// order (those of one instruction do if LDS takes its lanes one after the other), the waves take turns.
template <typename Item>
__device__ __forceinline__ void list_bucket(const ListJob& job, int bucket, uint32_t first, int n,
                                            const Item* __restrict__ items, Item* sorted, uint16_t* places, uint32_t* counts,
                                            uint32_t* wave_word) {
    const int tid = (int)threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const int n_here = 1 << job.low_bits;
    const int words = list_nodes(job.low_bits) / 4;  // of a wave's counts
    const uint32_t query_mask = (1u << job.query_bits) - 1u;
    const int rounds = (n + kListThreads - 1) / kListThreads;
    const int base = wave * rounds * kWave + lane;
    uint32_t* own = counts + wave * words;
    auto offsets_out = [&]() {
        const int64_t node0 = (int64_t)bucket << job.low_bits;
        for (int low = tid; low < n_here; low += kListThreads)
            if (node0 + low <= job.n_nodes) job.inc_off[node0 + low] = (int64_t)first + places[low];
    };
    Item x[kListRounds];
#pragma unroll
    for (int r = 0; r < kListRounds; ++r)
        if (r < rounds) x[r] = items[min(base + r * kWave, n - 1)];
#pragma unroll
    for (int r = 0; r < kListRounds; ++r) {
        if (r < rounds) {
            const uint32_t low = job.low_of(x[r]);
            if (base + r * kWave < n) atomicAdd(&own[low >> 2], 1u << ((low & 3u) * 8u));
        }
    }
    __syncthreads();
    // four nodes at a time: sums over the waves before, and pairs of all waves
    uint32_t sum = 0, most = 0;
    const int per = (words + kListThreads - 1) / kListThreads;
    for (int u = 0; u < per; ++u) {
        const int t = tid * per + u;
        if (t >= words) break;
        uint32_t even = 0, odd = 0;  // nodes 0 and 2, 1 and 3, 16 bits each
#pragma unroll
        for (int w = 0; w < kListWaves; ++w) {
            const uint32_t c = counts[w * words + t];
            counts[w * words + t] = even | odd << 8;
            even += c & 0x00FF00FFu;
            odd += c >> 8 & 0x00FF00FFu;
        }
        most |= (even | odd) & 0xFF00FF00u;  // more than a byte holds
        uint16_t* to = places + 4 * t;
        to[0] = (uint16_t)even;
        to[1] = (uint16_t)odd;
        to[2] = (uint16_t)(even >> 16);
        to[3] = (uint16_t)(odd >> 16);
        sum += (even & 0xFFFFu) + (even >> 16) + (odd & 0xFFFFu) + (odd >> 16);
    }
    const uint32_t incl = wave_incl_sum(sum);
    if (lane == kWave - 1) wave_word[wave] = incl;
    bool in_turns = __syncthreads_or(most != 0u) != 0;
    uint32_t before = incl - sum, all = 0;
    for (int w = 0; w < kListWaves; ++w) {
        if (w < wave) before += wave_word[w];
        all += wave_word[w];
    }
    in_turns = in_turns || all != (uint32_t)n;  // a byte ran over into its neighbour: 255 or 256 are missing
    if (!in_turns) {
        for (int u = 0; u < per; ++u) {
            const int t = tid * per + u;
            if (t >= words) break;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t here = places[4 * t + e];
                places[4 * t + e] = (uint16_t)before;
                before += here;
            }
        }
        __syncthreads();
        offsets_out();
#pragma unroll
        for (int r = 0; r < kListRounds; ++r) {
            if (r < rounds) {
                const uint32_t low = job.low_of(x[r]);
                if (base + r * kWave < n) {
                    const uint32_t shift = (low & 3u) * 8u;
                    const uint32_t rank = atomicAdd(&own[low >> 2], 1u << shift) >> shift & 0xFFu;
                    sorted[places[low] + rank] = x[r];
                }
            }
        }
        __syncthreads();
        bool wrong = false;
#pragma unroll 4
        for (int i = tid; i < n; i += kListThreads) {
            const Item item = sorted[i];
            wrong = wrong || item > sorted[min(i + 1, n - 1)];
            job.inc_q[first + i] = (int32_t)((uint32_t)item & query_mask);
        }
        in_turns = __syncthreads_or(wrong) != 0;
    }
    if (in_turns) {
        uint32_t word[kListRounds], place[kListRounds];
        __syncthreads();  // the words in front may still be read
        for (int t = tid; t < list_nodes(job.low_bits); t += kListThreads) counts[t] = 0u;
        __syncthreads();
        list_ranks<Item, kListThreads, kListRounds>(job, items, n, word, counts);
        list_node_places<kListThreads>(n_here, 0u, counts, wave_word, [&](int x, uint32_t place) {
            const int64_t node = ((int64_t)bucket << job.low_bits) + x;
            if (node <= job.n_nodes) job.inc_off[node] = (int64_t)first + place;
        });
        list_turns<kListThreads, kListRounds>(n, word, counts, place);
        uint32_t* queries = reinterpret_cast<uint32_t*>(sorted);
        const int shares = list_rounds<kListThreads>(n);
        int at = wave * shares * kWave + lane;
        asm volatile("" : "+v"(at));  // (no comparison of the loops above is kept for this one)
#pragma unroll
        for (int r = 0; r < kListRounds; ++r)
            if (r < shares && at + r * kWave < n) queries[place[r]] = (uint32_t)items[at + r * kWave] & query_mask;
        __syncthreads();
#pragma unroll 4
        for (int i = tid; i < n; i += kListThreads) job.inc_q[first + i] = (int32_t)queries[i];
    }
}

// Workgroups below n_buckets: a bucket each.  Those behind them: the nodes of the large buckets' chunks.
template <typename Item>
__global__ __launch_bounds__(kListThreads) void incidence_lists_kernel(ListJob job) {
    extern __shared__ __align__(16) unsigned char dynamic[];
    __shared__ uint32_t wave_word[kListWaves];
    __shared__ ListChunk chunk;
    const int n_nodes = list_nodes(job.low_bits);
    Item* sorted = reinterpret_cast<Item*>(dynamic);
    uint16_t* places = reinterpret_cast<uint16_t*>(dynamic + kListPairs * sizeof(Item));
    uint32_t* words = reinterpret_cast<uint32_t*>(places + n_nodes);
    const Item* items = static_cast<const Item*>(job.items);
    if ((int)blockIdx.x >= job.n_buckets) {
        list_chunk_counts<Item>(job, (int)blockIdx.x - job.n_buckets, (int)gridDim.x - job.n_buckets, words, &chunk,
                                wave_word);
        return;
    }
    const int b = (int)blockIdx.x;
    const uint32_t first = job.start_of(b), n = job.size_of(b);
    if (n > (uint32_t)kListPairs) return;
    uint4* clear = reinterpret_cast<uint4*>(words);
    for (int x = (int)threadIdx.x; x < n_nodes / 4; x += kListThreads) clear[x] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    list_bucket(job, b, first, (int)n, items + first, sorted, places, words, wave_word);
}

// LDS of a workgroup that puts chunks in order: two words a pair of a part (before that, two a node) and two a
// node.
size_t chunk_lds_bytes(int low_bits) {
    static_assert(kPartPairs >= 1 << kListBits, "room for the nodes' words");
    return 2 * (kPartPairs + (size_t)list_nodes(low_bits)) * sizeof(uint32_t);
}

// Puts the chunks of large buckets in order, a part that LDS holds at a time.  A chunk's places come from the
// counts of all chunks of its bucket; the bucket's first chunk also writes the nodes' offsets.
template <typename Item>
__global__ __launch_bounds__(kChunkThreads) void incidence_chunks_kernel(ListJob job) {
    extern __shared__ __align__(16) uint32_t chunk_words[];
    __shared__ uint32_t wave_word[kChunkWaves];
    __shared__ ListChunk shared;
    const int tid = (int)threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const int n_nodes = list_nodes(job.low_bits), n_here = 1 << job.low_bits;
    const uint32_t query_mask = (1u << job.query_bits) - 1u;
    uint32_t* queries = chunk_words;
    uint32_t* targets = queries + kPartPairs;
    uint32_t* all = queries;     // pairs of the bucket's nodes
    uint32_t* before = targets;  // of them, those in front of the chunk
    uint32_t* words = targets + kPartPairs;
    uint32_t* next = words + n_nodes;  // where a node's next pair goes in the output; less its place in the part
#pragma unroll 1
    for (int id = (int)blockIdx.x;; id += (int)gridDim.x) {
        const ListChunk c = list_chunk<kChunkThreads>(job, id, &shared, wave_word);
        if (c.bucket < 0) return;
        for (int x = tid; x < n_nodes; x += kChunkThreads) all[x] = before[x] = 0u;
        __syncthreads();
        // rows of 8 nodes in 16 bytes, as many rows at a time as there are threads for (with no more than
        // kListFlight a thread: a word takes its additions one after the other)
        const int pieces = n_nodes / 8, mine = c.at - c.bucket_chunk;
        const int groups = min(kChunkThreads / pieces, (c.n_bucket_chunks + kListFlight - 1) / kListFlight);
        const int group = tid / pieces, piece = tid & (pieces - 1);
        const uint4* counts =
            reinterpret_cast<const uint4*>(job.chunk_counts) + (int64_t)c.bucket_chunk * pieces + piece;
        uint32_t sum[8] = {}, in_front[8] = {};
#pragma unroll 1
        for (int k0 = group < groups ? group : c.n_bucket_chunks; k0 < c.n_bucket_chunks; k0 += groups * kListFlight) {
            uint4 v[kListFlight];
#pragma unroll
            for (int k = 0; k < kListFlight; ++k)
                v[k] = counts[(int64_t)min(k0 + k * groups, c.n_bucket_chunks - 1) * pieces];
#pragma unroll
            for (int k = 0; k < kListFlight; ++k) {
                const uint32_t w[4] = {v[k].x, v[k].y, v[k].z, v[k].w};
                const bool there = k0 + k * groups < c.n_bucket_chunks, first = k0 + k * groups < mine;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const uint32_t one = there ? w[e / 2] >> (e & 1) * 16 & 0xFFFFu : 0u;
                    sum[e] += one;
                    in_front[e] += first ? one : 0u;
                }
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if (sum[e] != 0u) atomicAdd(&all[piece * 8 + e], sum[e]);
            if (in_front[e] != 0u) atomicAdd(&before[piece * 8 + e], in_front[e]);
        }
        list_node_places<kChunkThreads>(n_here, job.start_of(c.bucket), all, wave_word, [&](int x, uint32_t place) {
            const int64_t node = ((int64_t)c.bucket << job.low_bits) + x;
            if (mine == 0 && node <= job.n_nodes) job.inc_off[node] = (int64_t)place;
            next[x] = place + before[x];
        });
#pragma unroll 1
        for (uint32_t part = 0; part < c.n; part += kPartPairs) {
            const Item* items = static_cast<const Item*>(job.items) + c.first + part;
            const int n = (int)min((uint32_t)kPartPairs, c.n - part), rounds = list_rounds<kChunkThreads>(n);
            const int base = wave * rounds * kWave + lane;
            for (int x = tid; x < n_nodes; x += kChunkThreads) words[x] = 0u;
            __syncthreads();
            uint32_t word[kPartRounds], place[kPartRounds];
            list_ranks<Item, kChunkThreads, kPartRounds>(job, items, n, word, words);
            list_node_places<kChunkThreads>(n_here, 0u, words, wave_word, [&](int x, uint32_t at) { next[x] -= at; });
            list_turns<kChunkThreads, kPartRounds>(n, word, words, place);
#pragma unroll
            for (int r = 0; r < kPartRounds; ++r) {
                if (r < rounds && base + r * kWave < n) {
                    const Item x = items[base + r * kWave];
                    queries[place[r]] = (uint32_t)x & query_mask;
                    targets[place[r]] = place[r] + next[job.low_of(x)];
                }
            }
            __syncthreads();
            for (int x = tid; x < n_here; x += kChunkThreads) next[x] += words[x];
#pragma unroll 4
            for (int i = tid; i < n; i += kChunkThreads) {
                const uint32_t to = targets[i];
                // (inside the output unless the list changes while it is sorted)
                if (to < (uint32_t)job.n) job.inc_q[to] = (int32_t)queries[i];
            }
            __syncthreads();
        }
    }
}

int sort_items(int64_t n) { return n <= kSortFew ? kSortFewItems : kSortMostItems; }
int64_t sort_tiles(int64_t n) {
    const int64_t tile = (int64_t)kSortThreads * sort_items(n);
    return (n + tile - 1) / tile;
}
size_t padded(size_t bytes) { return (bytes + 255) / 256 * 256; }

// Bits that hold 0 .. most.
int bits_of(uint64_t most) {
    int bits = 1;
    while (bits < 64 && (most >> bits) != 0) ++bits;
    return bits;
}

// Pairs of a bucket on average, at most: of more, not all buckets of a list that names all nodes alike
// would fit LDS.  In us, by buckets / 8 bits a pass: 3.1 M pairs on 2.9M nodes (4,443 a bucket) 52 / 108, on
// 600,000 50 / 106, 8.4 M on 2.9M (11,848) 387 / 205; 2.1 M on 10M nodes (8 bits only) 100, on 8M 80 / 100.
// (Lists that crowd, by buckets / 8 bits a pass: above.  Only where hardly another node is named, on graphs whose
// buckets have 8,192 nodes, or in short lists on small ones, do they take longer by buckets: 2.1 M pairs on 8M
// nodes, all with one node 159 / 127, half of them 133 / 136; 100,000 on 30,000 nodes, all with one 37 / 32, half
// 34 / 40; 2 M on 3,000 neighbours of 30,000 nodes 73 / 66.)
constexpr int64_t kBucketMean = 5500;

// Pairs of a chunk: where all pairs crowd in a few buckets there is a chunk a compute unit, or not quite (a
// bucket's last one is not full), and no fewer pairs than nodes that they are counted by (524,288 pairs with one
// of 2.9M nodes: 67 us with 4,096, 73 with 3,072); more than LDS takes at a time in whole parts (3.8 M pairs with
// one of 2.9M nodes 145 us, in chunks of a part 221).
uint32_t list_chunk_pairs(int64_t n, int low_bits) {
    const int64_t whole = n > (int64_t)kListChunks * 7 / 8 * kPartPairs ? kPartPairs : kChunkThreads;
    const int64_t pairs = (n / (kListChunks * 7 / 8) + whole) / whole * whole;
    return (uint32_t)(pairs < list_nodes(low_bits) ? list_nodes(low_bits) : pairs);
}
static_assert(kBuckets * kBucketMean / (kListChunks * 7 / 8) + kPartPairs < 1 << 16, "16 bits count a chunk's pairs");

// How a query list is sorted, and where its arrays lie in the scratch memory.
struct SortPlan {
    bool buckets;              // by buckets, or 8 bits a pass
    int64_t n_tiles;
    int items;                 // pairs of a thread of a tile
    int low_bits, query_bits;  // of an item of a bucket
    uint32_t chunk_pairs;
    size_t pairs[2], keys, item_at, hist, places, any_large, chunk_counts, bytes;
};
SortPlan sort_plan(int64_t n, int32_t k, int32_t n_nodes) {
    SortPlan p{};
    if (n < 1) n = 1;
    p.n_tiles = sort_tiles(n);
    p.items = sort_items(n);
    const int key_bits = bits_of((uint64_t)n_nodes);  // keys are 0..n_nodes
    p.low_bits = key_bits > kBucketBits ? key_bits - kBucketBits : 0;
    const int64_t n_buckets = (n_nodes >> p.low_bits) + 1;
    // (one pass of 8 bits: 64 pairs on 16 nodes 13 us, by buckets 17; 500,000 on 100 nodes 22 and 36)
    p.buckets = key_bits > 8 && key_bits <= kBucketBits + kListBits && n <= n_buckets * kBucketMean;
    auto part = [&](size_t bytes) {
        const size_t at = p.bytes;
        p.bytes += padded(bytes);
        return at;
    };
    if (p.buckets) {
        p.query_bits = bits_of((uint64_t)((n - 1) / k));
        p.chunk_pairs = list_chunk_pairs(n, p.low_bits);
        p.any_large = part(sizeof(uint32_t));
        p.item_at = part((size_t)n * (p.low_bits + p.query_bits <= 32 ? 4 : 8));
        // a large bucket has more than kListPairs pairs, and one chunk at most that is not full
        const int64_t large = n / kListPairs < kBuckets ? n / kListPairs : kBuckets;
        p.chunk_counts = part((size_t)(n / p.chunk_pairs + large) * list_nodes(p.low_bits) * sizeof(uint16_t));
    } else {
        p.pairs[0] = part((size_t)n * sizeof(uint2));
        p.pairs[1] = part((size_t)n * sizeof(uint2));
        p.keys = part((size_t)n * sizeof(uint32_t));
    }
    const size_t counts = (size_t)p.n_tiles * (p.buckets ? kBuckets : kSortBins) * sizeof(uint32_t);
    p.hist = part(counts);
    p.places = part(counts);
    return p;
}

// One pass: the pairs of `src` by kBins digits, to where `target` says.
template <int kItems, int kBins>
hipError_t sort_pass(hipStream_t stream, const SortPlan& p, const SortSource& src, int64_t n, int shift,
                     uint32_t* hist, uint32_t* places, const SortTarget& target, SmallScan* ss,
                     uint32_t spin_limit, uint32_t* any_large) {
    const dim3 grid((unsigned)p.n_tiles), block(kSortThreads);
    const size_t lds_bytes = (size_t)kSortThreads * kItems * sizeof(uint2);
    if (lds_bytes > 48 * 1024) {
        hipError_t rc = hipFuncSetAttribute(reinterpret_cast<const void*>(sort_scatter_kernel<kItems, kBins, kBins == kBuckets>),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (rc != hipSuccess) return rc;
    }
    sort_hist_kernel<kItems, kBins><<<grid, block, 0, stream>>>(src, n, shift, hist, any_large);
    sort_places_kernel<kBins><<<dim3(kBins / kWave), block, 0, stream>>>(
        hist, p.n_tiles, places, ss, spin_limit, (uint32_t)kListPairs, any_large);
    sort_scatter_kernel<kItems, kBins, kBins == kBuckets><<<grid, block, lds_bytes, stream>>>(src, n, shift, places, target);
    return hipGetLastError();
}

template <typename Item>
hipError_t launch_lists(hipStream_t stream, const ListJob& job) {
    const size_t lds_bytes = list_lds_bytes<Item>(job.low_bits);
    hipError_t rc = hipFuncSetAttribute(reinterpret_cast<const void*>(incidence_lists_kernel<Item>),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
    if (rc != hipSuccess) return rc;
    // no bucket of a shorter list is a large one
    const bool chunks = job.n > kListPairs;
    incidence_lists_kernel<Item><<<dim3((unsigned)(job.n_buckets + (chunks ? kListChunks : 0))), dim3(kListThreads),
                                   lds_bytes, stream>>>(job);
    if (!chunks) return hipGetLastError();
    const size_t chunk_bytes = chunk_lds_bytes(job.low_bits);
    rc = hipFuncSetAttribute(reinterpret_cast<const void*>(incidence_chunks_kernel<Item>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)chunk_bytes);
    if (rc != hipSuccess) return rc;
    incidence_chunks_kernel<Item><<<dim3(kListChunks), dim3(kChunkThreads), chunk_bytes, stream>>>(job);
    return hipGetLastError();
}

}  // namespace

size_t incidence_scratch_bytes(int64_t n_queries, int32_t k, int32_t n_nodes) {
    return sort_plan(n_queries * k, k, n_nodes).bytes;
}

hipError_t launch_query_incidence(hipStream_t stream, const int32_t* queries, int64_t n_queries,
                                  int32_t k, int32_t n_nodes, int64_t* inc_off, int32_t* inc_q,
                                  void* scratch, void* small_scan, uint32_t spin_limit,
                                  uint32_t* err) {
    const int64_t n = n_queries * k;
    const int offset_items = offsets_items(n_nodes);
    const dim3 offset_grid((unsigned)((int64_t)n_nodes / (kOffsetsThreads * offset_items) + 1));
    if (n == 0) {  // no entries: every part is empty
        incidence_offsets_kernel<<<offset_grid, dim3(kOffsetsThreads), 0, stream>>>(
            nullptr, 0, n_nodes, offset_items, inc_off);
        return hipGetLastError();
    }
    const SortPlan p = sort_plan(n, k, n_nodes);
    char* base = static_cast<char*>(scratch);
    uint32_t* hist = reinterpret_cast<uint32_t*>(base + p.hist);
    uint32_t* places = reinterpret_cast<uint32_t*>(base + p.places);
    SmallScan* ss = static_cast<SmallScan*>(small_scan);
    const bool few = p.items == kSortFewItems;
    if (p.buckets) {
        const SortSource src{queries, k, n_nodes, nullptr, err};
        const SortTarget target{nullptr, nullptr, nullptr, base + p.item_at, p.low_bits, p.query_bits};
        uint32_t* any_large = reinterpret_cast<uint32_t*>(base + p.any_large);
        hipError_t rc = few ? sort_pass<kSortFewItems, kBuckets>(stream, p, src, n, p.low_bits, hist, places,
                                                                 target, ss, spin_limit, any_large)
                            : sort_pass<kSortMostItems, kBuckets>(stream, p, src, n, p.low_bits, hist, places,
                                                                  target, ss, spin_limit, any_large);
        if (rc != hipSuccess) return rc;
        // the first tile's places are the buckets' starts
        const ListJob job{any_large, places, (n_nodes >> p.low_bits) + 1, n, target.items, p.low_bits, p.query_bits,
                          n_nodes, p.chunk_pairs, reinterpret_cast<uint16_t*>(base + p.chunk_counts),
                          inc_off, inc_q};
        return p.low_bits + p.query_bits <= 32 ? launch_lists<uint32_t>(stream, job)
                                               : launch_lists<uint64_t>(stream, job);
    }
    uint2* pairs[2] = {reinterpret_cast<uint2*>(base + p.pairs[0]), reinterpret_cast<uint2*>(base + p.pairs[1])};
    uint32_t* keys = reinterpret_cast<uint32_t*>(base + p.keys);
    const int key_bits = bits_of((uint64_t)n_nodes);
    for (int shift = 0, pass = 0; shift < key_bits; shift += 8, ++pass) {
        const bool last = shift + 8 >= key_bits;  // the last pass puts the queries where they belong
        const SortSource src{pass == 0 ? queries : nullptr, k, n_nodes, pairs[(pass + 1) & 1], err};
        const SortTarget target{pairs[pass & 1], last ? keys : nullptr, inc_q, nullptr, 0, 0};
        hipError_t rc = few ? sort_pass<kSortFewItems, kSortBins>(stream, p, src, n, shift, hist, places,
                                                                  target, ss, spin_limit, nullptr)
                            : sort_pass<kSortMostItems, kSortBins>(stream, p, src, n, shift, hist, places,
                                                                   target, ss, spin_limit, nullptr);
        if (rc != hipSuccess) return rc;
    }
    incidence_offsets_kernel<<<offset_grid, dim3(kOffsetsThreads), 0, stream>>>(
        keys, n, n_nodes, offset_items, inc_off);
    return hipGetLastError();
}

}  // namespace surel
