// The queries of every node (Sec. 3.6 "Mini-batching for Training": two nodes are neighbours
// when a query holds both, so the search walks node -> its queries -> their nodes).  Built by a
// stable radix sort of the (node, query) pairs of the query list: inc_q holds, node by node,
// the indices of the queries that name the node, ascending; inc_off[x] .. inc_off[x+1] is
// node x's part.
//
// The sort takes 8 bits a pass, least significant first, in three launches: digit counts of every
// tile, places (column sums over the tiles and over the digits), and the scatter, which puts a
// tile's pairs in order in LDS first, so that they leave as runs of a digit.  The first pass reads
// the query list itself.
// What bounds it: the memory round trips of the launches one after the other, at these sizes.
// A million two-node queries on 2.9M nodes: 86 us (three passes of 5 + 6 + 14, offsets 12); with
// a wavefront per tile of 1,024 pairs, a bisection per node and five launches a pass it was 290.
#include "device_util.h"
#include "kernels.h"
#include "small_scan.h"

namespace surel {

namespace {

constexpr int kSortThreads = 1024;
constexpr int kSortWaves = kSortThreads / kWave;
constexpr int kSortBins = 256;                    // 8 bits a pass
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
        return make_uint2(out ? (uint32_t)n_nodes : x, (uint32_t)(t / k));
    }
};

// hist[tile][d] = pairs of the tile whose key has digit d.
template <int kItems>
__global__ __launch_bounds__(kSortThreads) void sort_hist_kernel(SortSource src, int64_t n, int shift,
                                                                uint32_t* __restrict__ hist) {
    __shared__ uint32_t bins[kSortBins];
    const int tid = (int)threadIdx.x;
    if (tid < kSortBins) bins[tid] = 0u;
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
            atomicAdd(&bins[(pair[r].x >> shift) & (kSortBins - 1)], 1u);
    __syncthreads();
    if (tid < kSortBins) hist[(int64_t)blockIdx.x * kSortBins + tid] = bins[tid];
    raise_error(src.err, bad, kDevBadQuery);
}

// places[tile][d] = place of the tile's first pair with digit d.  A workgroup takes 64 digits, its
// 16 waves a share of the tiles each; the digits of the workgroups before it come in through
// small_scan.h (whose helpers read the counts at any time: the places are an array of their own).
constexpr int kPlaceGroups = kSortBins / kWave;
__global__ __launch_bounds__(kSortThreads) void sort_places_kernel(const uint32_t* __restrict__ hist,
                                                                  int64_t n_tiles,
                                                                  uint32_t* __restrict__ places,
                                                                  SmallScan* __restrict__ ss,
                                                                  uint32_t spin_limit) {
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
    uint32_t sum = 0;
    for (int64_t t = t0; t < t1; t += 8) {
        uint32_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = t + u < t1 ? column[(t + u) * kSortBins] : 0u;
#pragma unroll
        for (int u = 0; u < 8; ++u) sum += v[u];
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
        if (lane == kWave - 1) small_scan_publish(ss, (int)blockIdx.x, tag, incl);
        const int64_t base =
            small_scan_before(ss, (int)blockIdx.x, tag, spin_limit, lane, [&](int j) {
                uint32_t pairs = 0;  // of another workgroup's digits
#pragma unroll 1
                for (int64_t t = 0; t < n_tiles; ++t) pairs += hist[t * kSortBins + j * kWave + lane];
                return wave_bcast_u32(wave_incl_sum(pairs), kWave - 1);
            });
        if (lane == 0) {
            small_scan_done(ss, (int)blockIdx.x, tag, (int)gridDim.x);
            s_base = base;
        }
    }
    __syncthreads();
    uint32_t at = (uint32_t)s_base + incl - total + before;
    for (int64_t t = t0; t < t1; t += 8) {
        uint32_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = t + u < t1 ? column[(t + u) * kSortBins] : 0u;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (t + u < t1) to[(t + u) * kSortBins] = at;
            at += v[u];
        }
    }
}

// Moves a tile's pairs to their places.  Wave w owns the tile's pairs [w * 64 * kItems, ..) in
// rounds of 64, in index order: a pair's rank among the earlier ones of its digit is that of its
// wave so far, plus the lanes before it with the same digit (found by eight ballots).  keys / vals
// null: the pairs go to out_pairs, else (last pass) apart.
template <int kItems>
__global__ __launch_bounds__(kSortThreads) void sort_scatter_kernel(
    SortSource src, int64_t n, int shift, const uint32_t* __restrict__ places,
    uint2* __restrict__ out_pairs, uint32_t* __restrict__ keys, int32_t* __restrict__ vals) {
    __shared__ uint16_t count[kSortWaves][kSortBins];  // pairs of a digit in a wave, then before it
    __shared__ uint32_t start[kSortBins];              // first place of a digit inside the tile
    __shared__ uint32_t shift_to[kSortBins];           // its place in the output minus that
    __shared__ uint32_t wave_sum[kSortBins / kWave];
    extern __shared__ __align__(16) uint2 sorted[];    // the tile's pairs, in order
    const int tid = (int)threadIdx.x;
    const int lane = lane_id();
    const int wave = tid >> 6;
    for (int d = lane; d < kSortBins; d += kWave) count[wave][d] = 0;
    const int64_t tile = (int64_t)blockIdx.x * kSortThreads * kItems;
    const int64_t base = tile + wave * (kWave * kItems);
    uint2 pair[kItems];
    uint32_t rank[kItems];
    bool bad = false;
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const int64_t t = base + r * kWave + lane;
        pair[r] = t < n ? src.get(t, &bad) : make_uint2(0u, 0u);
    }
    wave_sync();
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const bool valid = base + r * kWave + lane < n;
        const uint32_t d = (pair[r].x >> shift) & (kSortBins - 1);
        uint64_t same = __ballot(valid);  // lanes whose pair has this lane's digit
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const uint64_t has = __ballot((d >> b) & 1u);
            same &= ((d >> b) & 1u) ? has : ~has;
        }
        const uint32_t in_round = (uint32_t)__popcll(same & below);
        const uint32_t group = (uint32_t)__popcll(same);
        const uint32_t so_far = count[wave][d];
        rank[r] = so_far + in_round;
        wave_sync();  // every lane has read the count before the group's last lane moves it on
        if (valid && in_round + 1 == group) count[wave][d] = (uint16_t)(so_far + group);
        wave_sync();
    }
    __syncthreads();
    uint32_t total = 0;
    if (tid < kSortBins) {
#pragma unroll
        for (int w = 0; w < kSortWaves; ++w) {
            const uint32_t c = count[w][tid];
            count[w][tid] = (uint16_t)total;
            total += c;
        }
    }
    uint32_t incl = 0;
    if (wave < kSortBins / kWave) {
        incl = wave_incl_sum(total);
        if (lane == kWave - 1) wave_sum[wave] = incl;
    }
    __syncthreads();
    if (tid < kSortBins) {
        uint32_t first = incl - total;
        for (int w = 0; w < wave; ++w) first += wave_sum[w];
        start[tid] = first;
        shift_to[tid] = places[(int64_t)blockIdx.x * kSortBins + tid] - first;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        if (base + r * kWave + lane < n) {
            const uint32_t d = (pair[r].x >> shift) & (kSortBins - 1);
            sorted[start[d] + count[wave][d] + rank[r]] = pair[r];
        }
    }
    __syncthreads();
    const int n_here = (int)min((int64_t)kSortThreads * kItems, n - tile);
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const int i = r * kSortThreads + tid;
        if (i < n_here) {
            const uint2 p = sorted[i];
            const uint32_t to = shift_to[(p.x >> shift) & (kSortBins - 1)] + (uint32_t)i;
            if (keys == nullptr) {
                out_pairs[to] = p;
            } else {
                keys[to] = p.x;
                vals[to] = (int32_t)p.y;
            }
        }
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

int sort_items(int64_t n) { return n <= kSortFew ? kSortFewItems : kSortMostItems; }
int64_t sort_tiles(int64_t n) {
    const int64_t tile = (int64_t)kSortThreads * sort_items(n);
    return (n + tile - 1) / tile;
}
size_t padded(size_t bytes) { return (bytes + 255) / 256 * 256; }

}  // namespace

size_t incidence_scratch_bytes(int64_t n_entries) {
    const int64_t n = n_entries > 0 ? n_entries : 1;
    return 2 * padded((size_t)n * sizeof(uint2)) + padded((size_t)n * sizeof(uint32_t)) +
           2 * padded((size_t)sort_tiles(n) * kSortBins * sizeof(uint32_t));
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
    const int64_t n_tiles = sort_tiles(n);
    const int items = sort_items(n);
    char* p = static_cast<char*>(scratch);
    uint2* pairs[2] = {reinterpret_cast<uint2*>(p), reinterpret_cast<uint2*>(p + padded((size_t)n * sizeof(uint2)))};
    p += 2 * padded((size_t)n * sizeof(uint2));
    uint32_t* keys = reinterpret_cast<uint32_t*>(p);
    p += padded((size_t)n * sizeof(uint32_t));
    uint32_t* hist = reinterpret_cast<uint32_t*>(p);
    p += padded((size_t)n_tiles * kSortBins * sizeof(uint32_t));
    uint32_t* places = reinterpret_cast<uint32_t*>(p);

    int bits = 1;  // keys are 0..n_nodes
    while (bits < 32 && ((uint32_t)n_nodes >> bits) != 0u) ++bits;
    const dim3 grid((unsigned)n_tiles), block(kSortThreads);
    const size_t lds_bytes = (size_t)kSortThreads * items * sizeof(uint2);
    if (items == kSortMostItems) {
        hipError_t rc = hipFuncSetAttribute(
            reinterpret_cast<const void*>(sort_scatter_kernel<kSortMostItems>),
            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (rc != hipSuccess) return rc;
    }
    for (int shift = 0, pass = 0; shift < bits; shift += 8, ++pass) {
        const bool last = shift + 8 >= bits;  // the last pass puts the queries where they belong
        const SortSource src{pass == 0 ? queries : nullptr, k, n_nodes, pairs[(pass + 1) & 1], err};
        uint2* to = pairs[pass & 1];
        if (items == kSortMostItems) {
            sort_hist_kernel<kSortMostItems><<<grid, block, 0, stream>>>(src, n, shift, hist);
        } else {
            sort_hist_kernel<kSortFewItems><<<grid, block, 0, stream>>>(src, n, shift, hist);
        }
        sort_places_kernel<<<dim3(kPlaceGroups), block, 0, stream>>>(
            hist, n_tiles, places, static_cast<SmallScan*>(small_scan), spin_limit);
        if (items == kSortMostItems) {
            sort_scatter_kernel<kSortMostItems><<<grid, block, lds_bytes, stream>>>(
                src, n, shift, places, to, last ? keys : nullptr, inc_q);
        } else {
            sort_scatter_kernel<kSortFewItems><<<grid, block, lds_bytes, stream>>>(
                src, n, shift, places, to, last ? keys : nullptr, inc_q);
        }
    }
    incidence_offsets_kernel<<<offset_grid, dim3(kOffsetsThreads), 0, stream>>>(
        keys, n, n_nodes, offset_items, inc_off);
    return hipGetLastError();
}

}  // namespace surel
