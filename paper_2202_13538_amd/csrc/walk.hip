// Walk sampling (Sec. 3.2 "Walk Sampling"; Algorithm 1, walk step).
//
// One wavefront per seed; a lane moves two walks at a time (two independent gathers in
// flight per lane), ceil(M/128) passes.  A pass keeps its 128
// walks in LDS ([walk][position]) and then streams them out as one contiguous block, so
// the global stores are full-width instead of lane-strided.  Walk rows are written with
// non-temporal stores: they are not read again by this kernel and should not push the
// graph out of the caches that serve the neighbour gathers.
//
// Neighbour records.  A step needs the chosen neighbour's id and then that neighbour's own
// row (start, degree) for the next step: two dependent gathers that each miss the L2 and
// pull a whole cache line for a few bytes, which is what bounds this kernel.  When the job
// is large next to the graph, a small kernel first expands the CSR into one record per edge
// entry, (neighbour id, its row start, its degree), so that every step after the first is a
// single gather: one 64-bit word, or 16 bytes where ids and row starts leave the degree too few of
// its bits (walk_core.h).  All forms make exactly the same walks.
//
// Optionally the kernel also reports |V_u|, the number of distinct nodes of each seed's
// walks (Algorithm 1: V_u = set(W_u)), through an LDS hash set fed while the walkers move.
// The kernel waits on memory nearly all the time, so this costs little, and it saves the
// RPE builder a counting pass over the walks.
#include "device_util.h"
#include "distinct.h"
#include "kernels.h"
#include "walk_core.h"
#include "walk_table.h"

namespace surel {

// Rows of 12 consecutive nodes in 16 bytes: the start of the first row, then the degrees, a byte
// each.  A byte of 255 says "ask row_ptr": a degree that does not fit, a malformed row, and every
// row behind such a one in the group (a row starts where the degrees before it in the group end).
constexpr int kRowsPerGroup = 12;
constexpr uint32_t kAskRowPtr = 255u;
static size_t row_group_bytes(int32_t n_nodes) {
    return ((size_t)n_nodes + kRowsPerGroup - 1) / kRowsPerGroup * sizeof(uint4);
}

__global__ void row_group_kernel(const int32_t* __restrict__ row_ptr, int32_t n_nodes,
                                 int64_t n_edges, uint4* __restrict__ groups) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t x0 = g * kRowsPerGroup;
    if (x0 >= n_nodes) return;
    int32_t start[kRowsPerGroup + 1];
#pragma unroll
    for (int j = 0; j <= kRowsPerGroup; ++j) start[j] = row_ptr[min(x0 + j, (int64_t)n_nodes)];
    uint32_t w[4] = {(uint32_t)start[0]};
    bool ask = false;
#pragma unroll
    for (int j = 0; j < kRowsPerGroup; ++j) {
        const int32_t lo = start[j], hi = start[j + 1];
        ask = ask || lo < 0 || hi < lo || (int64_t)hi > n_edges || (uint32_t)(hi - lo) >= kAskRowPtr;
        w[1 + j / 4] |= (ask ? kAskRowPtr : (uint32_t)(hi - lo)) << (j % 4 * 8);
    }
    groups[g] = make_uint4(w[0], w[1], w[2], w[3]);
}

// The record of every CSR entry e (layouts in walk_core.h): the neighbour col_idx[e], the start
// of its row and its degree; an entry that names no node, or whose row is malformed, gets the
// layout's "bad entry" id (the walker will stay in place and flag it).
// kGroups: the rows are looked up in groups (above) instead of row_ptr, see rows_in_groups.  Entries
// and packed records go past the caches, which a pass's outputs have filled by then: 20 M entries on 1M
// nodes 137 us, 161 through the caches, 2.6 M on 235,000 22 and 24, 42 M on 524,288 249 and 286.
// (Only where nothing else had been written since the launch before were they faster through the
// caches, up to 24 M entries.)  Short records of a workgroup are whole words, put together from LDS.
// What bounds this kernel is the random look-up: a 128-byte line each, 56 G/s from memory where it
// misses the L2 and 260 G/s from an L2 with nothing else to do.  The 11.6 MB of row_ptr of a
// 2.9M-node graph miss a 4 MB L2 most of the time, its groups are 3.9 MB: 60 M entries in 508 us,
// 693 with two loads from row_ptr an entry.  Groups of 28 rows in 32 bytes are two requests: 569 us.
constexpr int kRecordThreads = 256;
constexpr int kRecordItems = 4;  // entries of a thread, all their look-ups in flight
template <int kRec, bool kGroups>
__global__ __launch_bounds__(kRecordThreads) void edge_record_kernel(
    const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx, int32_t n_nodes,
    int64_t n_edges, int id_bits, int lo_bits, const uint4* __restrict__ groups,
    void* __restrict__ rec) {
    const int64_t e0 = (int64_t)blockIdx.x * (kRecordThreads * kRecordItems) + threadIdx.x;
    uint32_t t[kRecordItems];
    bool node[kRecordItems];
#pragma unroll
    for (int u = 0; u < kRecordItems; ++u) {
        t[u] = (uint32_t)__builtin_nontemporal_load(col_idx + min(e0 + u * kRecordThreads, n_edges - 1));
    }
#pragma unroll
    for (int u = 0; u < kRecordItems; ++u) node[u] = t[u] < (uint32_t)n_nodes;
    int32_t lo[kRecordItems], hi[kRecordItems];
    if constexpr (kGroups) {
        uint4 a[kRecordItems];
        uint32_t j[kRecordItems];
#pragma unroll
        for (int u = 0; u < kRecordItems; ++u) {
            const uint32_t x = node[u] ? t[u] : 0u;
            const uint32_t g = x / kRowsPerGroup;
            j[u] = x - g * kRowsPerGroup;
            a[u] = groups[g];
        }
#pragma unroll
        for (int u = 0; u < kRecordItems; ++u) {
            const uint32_t w[3] = {a[u].y, a[u].z, a[u].w};
            // the word with the node's degree and what the degrees in front of it add up to
            uint32_t start = a[u].x, degrees = w[0], sum = a[u].x;
#pragma unroll
            for (uint32_t q = 1; q < 3; ++q) {
                sum = __builtin_amdgcn_sad_u8(w[q - 1], 0u, sum);
                const bool here = j[u] >= 4u * q;
                start = here ? sum : start;
                degrees = here ? w[q] : degrees;
            }
            const uint32_t in_front = 8u * (j[u] & 3u);
            start = __builtin_amdgcn_sad_u8(__builtin_amdgcn_ubfe(degrees, 0u, in_front), 0u, start);
            const uint32_t degree = __builtin_amdgcn_ubfe(degrees, in_front, 8u);
            lo[u] = (int32_t)start;
            hi[u] = (int32_t)(start + degree);
            if (node[u] && degree == kAskRowPtr) row_ends(row_ptr, t[u], &lo[u], &hi[u]);
        }
    } else {
#pragma unroll
        for (int u = 0; u < kRecordItems; ++u) row_ends(row_ptr, node[u] ? t[u] : 0u, &lo[u], &hi[u]);
    }
    if constexpr (kRec == kRecShort) {
        constexpr int kTile = kRecordThreads * kRecordItems;
        __shared__ uint32_t ids[kTile + 1];
        const int tid = (int)threadIdx.x;
        const int64_t first = (int64_t)blockIdx.x * kTile;
        const int n = (int)min((int64_t)kTile, n_edges - first);
#pragma unroll
        for (int u = 0; u < kRecordItems; ++u) {
            const bool ok = node[u] && lo[u] >= 0 && hi[u] >= lo[u] && (int64_t)hi[u] <= n_edges;
            const int i = u * kRecordThreads + tid;
            ids[i] = i >= n ? 0u : ok ? t[u] : (uint32_t)n_nodes;
        }
        __syncthreads();
        // a tile is 32 * id_bits words, and begins with a word of its own
        uint32_t* to = static_cast<uint32_t*>(rec) + (int64_t)blockIdx.x * (kTile / 32 * id_bits);
        const int n_words = (n * id_bits + 31) / 32;
        for (int j = tid; j < n_words; j += kRecordThreads) {
            int i = j * 32 / id_bits, at = i * id_bits - j * 32;  // the first id of word j, and its place there
            uint32_t word = ids[i] >> -at;
            for (at += id_bits; at < 32; at += id_bits) word |= ids[++i] << at;
            to[j] = word;
        }
        return;
    }
#pragma unroll
    for (int u = 0; u < kRecordItems; ++u) {
        const int64_t e = e0 + u * kRecordThreads;
        if (e >= n_edges) return;
        const bool ok = node[u] && lo[u] >= 0 && hi[u] >= lo[u] && (int64_t)hi[u] <= n_edges;
        if (kRec == kRecWide) {
            static_cast<int4*>(rec)[e] =
                ok ? make_int4((int)t[u], lo[u], hi[u] - lo[u], 0) : make_int4(-1, 0, 0, 0);
        } else {
            const uint32_t deg_big = (1u << rec_degree_bits(id_bits, lo_bits)) - 1u;
            unsigned long long r = (unsigned long long)(uint32_t)n_nodes;  // bad entry
            if (ok) {
                const uint32_t deg = min((uint32_t)(hi[u] - lo[u]), deg_big);
                r = (unsigned long long)t[u] | ((unsigned long long)(uint32_t)lo[u] << id_bits) |
                    ((unsigned long long)deg << (id_bits + lo_bits));
            }
            __builtin_nontemporal_store(r, static_cast<unsigned long long*>(rec) + e);
        }
    }
}

template <bool kCount, int kRec>
__global__ __launch_bounds__(kWalkWavesPerBlock* kWave) void walk_kernel(
    const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
    const void* __restrict__ rec, int id_bits, int lo_bits, int32_t n_nodes, int64_t n_edges,
    const int32_t* __restrict__ seeds, int64_t n_seeds, int32_t M, int32_t m, uint32_t key0,
    uint32_t key1, int32_t* __restrict__ walks, int32_t* __restrict__ set_sizes, int32_t slots,
    uint32_t* __restrict__ err) {
    extern __shared__ int32_t lds[];
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t i = (int64_t)blockIdx.x * kWalkWavesPerBlock + wave;
    if (i >= n_seeds) return;  // whole waves leave; no block-wide barrier is used below

    const int L = m + 1;
    const int per_wave = kWalkChains * kWave * L + (kCount ? slots : 0);
    int32_t* stage = lds + wave * per_wave;
    uint32_t* table = reinterpret_cast<uint32_t*>(stage + kWalkChains * kWave * L);
    int32_t* out_seed = walks + i * (int64_t)M * L;

    const int32_t u = __builtin_amdgcn_readfirstlane(seeds[i]);
    if (u < 0 || u >= n_nodes) {
        if (lane == 0) {
            atomicOr(err, kDevBadSeed);
            if (kCount) set_sizes[i] = 0;
        }
        const int total = M * L;
        for (int t = lane; t < total; t += kWave) __builtin_nontemporal_store(-1, out_seed + t);
        return;
    }

    int n_distinct = 0;
    if (kCount) {
        distinct_clear(table, slots, lane);
        wave_sync();
        n_distinct = distinct_insert(table, slots, (uint32_t)u, lane == 0);
    }

    const WalkGraph g{row_ptr, col_idx, rec, id_bits, lo_bits, n_nodes, n_edges};
    int32_t u_lo, u_deg;
    bool bad_graph = seed_row(g, u, &u_lo, &u_deg);
    for (int w0 = 0; w0 < M; w0 += kWalkChains * kWave) {
        int w[kWalkChains];
        bool active[kWalkChains];
        int32_t* row[kWalkChains];
#pragma unroll
        for (int c = 0; c < kWalkChains; ++c) {
            w[c] = w0 + c * kWave + lane;
            active[c] = w[c] < M;
            row[c] = stage + (c * kWave + lane) * L;
        }
        bad_graph |= walk_many<kRec, kWalkChains>(
            g, u, u_lo, u_deg, w, active, m, key0, key1, row, [&](int c, int32_t node) {
                if (kCount) n_distinct += distinct_insert(table, slots, (uint32_t)node, active[c]);
            });
        wave_sync();
        const int total = min(kWalkChains * kWave, M - w0) * L;
        int32_t* out = out_seed + (int64_t)w0 * L;
        for (int t = lane; t < total; t += kWave) __builtin_nontemporal_store(stage[t], out + t);
        wave_sync();
    }
    if (kCount && lane == 0) set_sizes[i] = n_distinct;
    raise_error(err, bad_graph, kDevBadGraph);
}

bool walks_want_records(int64_t n_edges, int64_t n_seeds, int32_t M, int32_t m) {
    // the expansion reads every edge entry once; it pays off when the steps after the first
    // outnumber the edge entries several times
    return m >= 2 && n_edges > 0 && n_seeds * (int64_t)M * (m - 1) >= 4 * n_edges;
}

static int bits_for(uint64_t max_value) {  // bits that hold 0 .. max_value
    int b = 1;
    while (b < 64 && (max_value >> b) != 0) b += 1;
    return b;
}

// Whether records are the ids alone: where row_ptr leaves the larger part of a 4 MB L2 to them and packed
// records are at least twice as large as it.  Walks + RPE (M = 100, m = 4 where nothing else is said), us,
// packed / short (up to 235,000 nodes short ones of whole bytes, then / of whole bits):
//    30,000 nodes   0.6 M entries, M = 200   193 /   195     1.2 M            130 /   114 /   114
//    60,000 nodes   0.6 M, M = 200           302 /   307     4.8 M, M = 200   671 /   485 /   485
//   100,000 nodes   1.2 M                    326 /   324     1.6 M, m = 9     742 /   562 /   520
//                   8 M, M = 200           1,154 / 1,034 / 955
//   235,000 nodes   2.6 M, M = 200         1,538 / 1,450 / 1,430   16 M, M = 200  2,721 / 2,668 / 2,570
//   300,000 nodes   4.8 M, M = 50            749 /   721
//   350,000 nodes   7 M, M = 50              940 /   923     3 M            1,138 / 1,086
//   500,000 nodes   2 M, M = 50              977 / 1,012     6 M, M = 50    1,152 / 1,206
// Walks alone, counting their sets: 320,000 nodes, 3 M, M = 150 1,540 / 1,147, 5 M, M = 150, m = 9 5,539 /
// 5,377, 14 M 6,600 / 6,632; 390,000, 8 M, M = 150 2,408 / 2,496.
// (Entries are addressed with 24 bits.)
// few_waves (walk_waves_are_few), M = 292, m = 6: 140,000 nodes, 1.4 M 2,371 / 2,166, 200,000, 8 M 4,659 / 4,390,
// 235,000, 2.6 M 4,151 / 4,428, 327,680, 3.2 M 5,686 / 6,271.  fused, past 2^18 nodes: 300,000, 10 M, M = 100,
// m = 3 1,054 / 987, M = 64, m = 9 3,201 / 3,227; 327,680, 14 M 1,242 / 1,203 and 3,600 / 3,749, M = 150, m = 5
// 3,775 / 3,854.
constexpr int32_t kShortNodes = 5 << 16, kShortNodesFewWaves = 200'000;
static bool rows_beside_short_records(int32_t n_nodes, int64_t n_edges, bool few_waves, bool fused) {
    return n_nodes <= (few_waves ? kShortNodesFewWaves : kShortNodes) && n_edges >= 1 << 20 &&
           n_edges < (fused && n_nodes > 1 << 18 ? 12'000'000 : 1 << 24);
}

EdgeRecords edge_record_plan(int32_t n_nodes, int64_t n_edges, bool few_waves, bool fused) {
    EdgeRecords plan;
    plan.id_bits = bits_for((uint64_t)n_nodes);   // n_nodes itself marks a bad entry
    plan.lo_bits = bits_for((uint64_t)n_edges);   // 31 at most
    // packed records where ordinary degrees fit their field, the wide layout otherwise.  (On
    // small graphs the packed array fits more of its lines into the L2s.)
    plan.format = rec_degree_bits(plan.id_bits, plan.lo_bits) >= 12 ? kRecPacked : kRecWide;
    if (rows_beside_short_records(n_nodes, n_edges, few_waves, fused)) plan.format = kRecShort;
    // the degree lies in the word's upper half
    if (plan.format == kRecPacked && plan.id_bits + plan.lo_bits < 32) plan.lo_bits = 32 - plan.id_bits;
    return plan;
}

// Whether the rows are worth grouping: where row_ptr outgrows a 4 MB L2 so far (5 MB and more) that
// the hot rows of a graph with uneven degrees do not stay there either, and where most entries name
// a node whose degree fits a byte.  Measured with cold caches, as the pass before leaves them, us,
// rows from row_ptr / grouped (the launch that groups them among it):
//                               entries a node, exponent of the degrees
//   nodes          4, 2.3        20, 2.1        20, 2.5        28, 2.3       20, even
//     700,000     23 /  28       90 / 108       90 / 100      123 / 145       90 /  95
//   1,000,000     31 /  36      135 / 153      136 / 142      188 / 205      136 / 132
//   1,200,000     39 /  41      172 / 184      175 / 168      240 / 248
//   1,500,000     50 /  49      222 / 238      228 / 209      312 / 321      235 / 197
//   2,000,000     75 /  63      327 / 342      369 / 291      491 / 459
//   2,900,000    133 /  94      596 / 540      682 / 465      916 / 730      717 / 392
constexpr int32_t kGroupNodes = 5 << 18;
static_assert(kGroupNodes > kShortNodes, "short records are not made from groups");
static bool rows_in_groups(int32_t n_nodes, int64_t n_edges) {
    return n_nodes >= kGroupNodes && n_edges <= 32 * (int64_t)n_nodes;
}

static size_t record_array_bytes(const EdgeRecords& plan, int64_t n_edges) {
    const size_t bits = plan.format == kRecShort ? plan.id_bits : plan.format == kRecPacked ? 64 : 128;
    // short records are read as the four bytes from where one begins: the last one's may end behind it
    const size_t behind = plan.format == kRecShort ? 4 : 0;
    return (((size_t)n_edges * bits + 7) / 8 + behind + 15) & ~(size_t)15;
}

size_t edge_record_bytes(const EdgeRecords& plan, int32_t n_nodes, int64_t n_edges) {
    return record_array_bytes(plan, n_edges) +
           (rows_in_groups(n_nodes, n_edges) ? row_group_bytes(n_nodes) : 0);
}

template <bool kCount, int kRec>
static hipError_t launch_walks_cfg(hipStream_t stream, const int32_t* row_ptr,
                                   const int32_t* col_idx, const EdgeRecords& rec, int32_t n_nodes,
                                   int64_t n_edges, const int32_t* seeds, int64_t n_seeds,
                                   int32_t M, int32_t m, uint64_t rng_seed, int32_t* walks,
                                   int32_t* set_sizes, uint32_t* err) {
    const int64_t blocks = (n_seeds + kWalkWavesPerBlock - 1) / kWalkWavesPerBlock;
    const int slots = !kCount ? 0 : kRec == kRecShort ? walk_table(M, m).slots : distinct_slots(1 + M * m);
    const size_t lds_bytes = (size_t)kWalkWavesPerBlock * (kWalkChains * kWave * (m + 1) + slots) * 4;
    if (lds_bytes > 48 * 1024) {
        hipError_t rc = hipFuncSetAttribute(
            reinterpret_cast<const void*>(walk_kernel<kCount, kRec>),
            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (rc != hipSuccess) return rc;
    }
    hipLaunchKernelGGL((walk_kernel<kCount, kRec>), dim3((unsigned)blocks),
                       dim3(kWalkWavesPerBlock * kWave), lds_bytes, stream, row_ptr, col_idx,
                       rec.data, rec.id_bits, rec.lo_bits, n_nodes, n_edges, seeds, n_seeds, M, m,
                       (uint32_t)(rng_seed & 0xFFFFFFFFull), (uint32_t)(rng_seed >> 32), walks,
                       set_sizes, slots, err);
    return hipGetLastError();
}

hipError_t launch_edge_records(hipStream_t stream, const int32_t* row_ptr, const int32_t* col_idx,
                               int32_t n_nodes, int64_t n_edges, const EdgeRecords& rec) {
    if (n_edges <= 0) return hipSuccess;
    const int64_t tile = kRecordThreads * kRecordItems;
    const dim3 grid((unsigned)((n_edges + tile - 1) / tile)), block(kRecordThreads);
    void* data = const_cast<void*>(rec.data);
    uint4* groups = nullptr;  // they lie behind the records
    if (rows_in_groups(n_nodes, n_edges)) {
        groups = reinterpret_cast<uint4*>(static_cast<char*>(data) + record_array_bytes(rec, n_edges));
        const int64_t n_groups = (int64_t)(row_group_bytes(n_nodes) / sizeof(uint4));
        row_group_kernel<<<dim3((unsigned)((n_groups + 63) / 64)), dim3(64), 0, stream>>>(
            row_ptr, n_nodes, n_edges, groups);
    }
    const auto kernel = rec.format == kRecShort
                            ? edge_record_kernel<kRecShort, false>  // of graphs too small for groups
                        : rec.format == kRecPacked
                            ? (groups ? edge_record_kernel<kRecPacked, true> : edge_record_kernel<kRecPacked, false>)
                            : (groups ? edge_record_kernel<kRecWide, true> : edge_record_kernel<kRecWide, false>);
    kernel<<<grid, block, 0, stream>>>(row_ptr, col_idx, n_nodes, n_edges, rec.id_bits, rec.lo_bits, groups,
                                       data);
    return hipGetLastError();
}

template <bool kCount>
static hipError_t launch_walks_c(hipStream_t stream, const int32_t* row_ptr, const int32_t* col_idx,
                                 const EdgeRecords& rec, int32_t n_nodes, int64_t n_edges,
                                 const int32_t* seeds, int64_t n_seeds, int32_t M, int32_t m,
                                 uint64_t rng_seed, int32_t* walks, int32_t* set_sizes,
                                 uint32_t* err) {
#define SUREL_WALK_ARGS \
    stream, row_ptr, col_idx, rec, n_nodes, n_edges, seeds, n_seeds, M, m, rng_seed, walks, set_sizes, err
    if (rec.data == nullptr) return launch_walks_cfg<kCount, kRecNone>(SUREL_WALK_ARGS);
    if (rec.format == kRecPacked) return launch_walks_cfg<kCount, kRecPacked>(SUREL_WALK_ARGS);
    if (rec.format == kRecShort) return launch_walks_cfg<kCount, kRecShort>(SUREL_WALK_ARGS);
    return launch_walks_cfg<kCount, kRecWide>(SUREL_WALK_ARGS);
}

hipError_t launch_walks(hipStream_t stream, const int32_t* row_ptr, const int32_t* col_idx,
                        int32_t n_nodes, int64_t n_edges, const int32_t* seeds, int64_t n_seeds,
                        int32_t M, int32_t m, uint64_t rng_seed, int32_t* walks,
                        int32_t* set_sizes, const EdgeRecords& rec, uint32_t* err) {
    if (n_seeds == 0) return hipSuccess;
    if (set_sizes != nullptr) return launch_walks_c<true>(SUREL_WALK_ARGS);
    return launch_walks_c<false>(SUREL_WALK_ARGS);
#undef SUREL_WALK_ARGS
}

}  // namespace surel
