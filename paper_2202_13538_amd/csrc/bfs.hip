// Mini-batches by breadth-first search over nodes that share queries (Sec. 3.6 "Mini-batching
// for Training"; Algorithm 2, the BFS step).  One workgroup (four wavefronts, or one for small
// batches) builds one mini-batch; a launch builds many (the iterations of Algorithm 2 draw their seed-sets independently).
//
// The search is the first-in first-out one: the node set V̄ is its own queue, a node's queries
// are taken in ascending index, a query's nodes in tuple order, and a query enters the batch
// together with all its nodes or ends the search.  The workgroup reproduces that order without
// walking the queue one node at a time: it takes the next stretch of the queue whose query
// lists hold at most a chunk of entries (1,024, fewer for small batches), numbers those
// entries ("candidates") in queue order,
// and lets every query keep the smallest candidate number that names it (atomic minimum in a
// hash table).  The candidates that kept their query are the newly reached queries, in the
// order the queue would have reached them; their nodes are numbered (query's place, position
// in the tuple) and settled the same way.  Prefix sums then give every new query and node its
// place, and the limits B1, B2 cut the stretch exactly where the queue would have stopped.
#include "device_util.h"
#include "kernels.h"

namespace surel {

namespace {

constexpr int kBfsPer = 4;        // candidates (or new queries) per thread, at most
constexpr int kBfsMaxThreads = 256;  // a workgroup has 256 threads, or 64 for small batches
constexpr int kBfsMaxChunk = kBfsMaxThreads * kBfsPer;  // candidates settled at a time, at most
// Searches whose tables fit into this much LDS keep them there: an insertion is a few LDS round trips instead
// of atomics that travel to memory.  8,192 searches of 32 queries: 71 us, with the tables in global memory
// 524.  Of a chunk's new queries only those that the batch has room for get their nodes entered, and what a
// thread alone needs of a chunk is in its registers: such a search's LDS is then 4.7 KB with the static
// part, four of the 128 parts that a compute unit's LDS is given out in, and 32 searches of a compute unit
// run at a time (which also takes no more scalar registers than eight waves of a SIMD have): 27 us (34 with
// 25 searches, lists of candidates in LDS and two loads of a query's nodes and of a list's place).
// Searches of more than 64 queries may have a compute unit's LDS for one of them: 1,024 queries of two
// nodes, 16 / 256 / 4,096 searches 40 / 48 / 551 us, with tables in global memory 90 / 176 / 2,087; 2,000
// queries 65 / 80 / 930 and 146 / 277 / 3,506.
constexpr size_t kBfsLdsMost = 79 * 1024;       // of a search of one wavefront
constexpr size_t kBfsLdsMostWide = 156 * 1024;  // of one of four, which has 3.1 KB that are not dynamic
constexpr size_t kBfsLdsEight = 16 * 1024;      // of one of four, eight of which a compute unit then holds
constexpr int kBfsMaxK = 3;
constexpr uint32_t kBfsEmpty = 0xFFFFFFFFu;

__device__ __forceinline__ uint32_t bfs_hash(uint32_t x) {
    x ^= x >> 16;
    x *= 0x7feb352du;
    x ^= x >> 15;
    x *= 0x846ca68bu;
    x ^= x >> 16;
    return x;
}

// A value read that sees what atomics of other waves have left in the table (kLds: the table lies
// in LDS, where a workgroup's barrier is all that takes).
template <bool kLds>
__device__ __forceinline__ uint32_t table_load(const uint32_t* p) {
    if constexpr (kLds) {
        return *p;
    } else {
        return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Open addressing over (key, value) pairs: finds or claims the slot of `key` and lowers its
// value to `val` if that is smaller.  Returns the slot, or kBfsEmpty if no slot was found
// within the table (cannot happen while the table is not full).
__device__ __forceinline__ uint32_t insert_min(uint32_t* tab, uint32_t mask, uint32_t key,
                                               uint32_t val) {
    uint32_t h = bfs_hash(key) & mask;
    for (uint32_t probe = 0; probe <= mask; ++probe) {
        const uint32_t seen = atomicCAS(&tab[2 * h], kBfsEmpty, key);
        if (seen == kBfsEmpty || seen == key) {
            atomicMin(&tab[2 * h + 1], val);
            return h;
        }
        h = (h + 1) & mask;
    }
    return kBfsEmpty;
}

// Exclusive prefix sum of one value per thread over the workgroup of T threads; *total = the sum.
template <int T>
__device__ __forceinline__ uint32_t bfs_block_scan(uint32_t v, uint32_t* total, uint32_t* wave_sums) {
    const int lane = lane_id();
    const int wave = threadIdx.x >> 6;
    const uint32_t incl = wave_incl_sum(v);
    if constexpr (T == kWave) {
        *total = wave_bcast_u32(incl, kWave - 1);
        return incl - v;
    }
    __syncthreads();  // wave_sums may still be read from the previous scan
    if (lane == kWave - 1) wave_sums[wave] = incl;
    __syncthreads();
    uint32_t base = 0, sum = 0;
#pragma unroll
    for (int w = 0; w < T / kWave; ++w) {
        if (w < wave) base += wave_sums[w];
        sum += wave_sums[w];
    }
    *total = sum;
    return base + incl - v;
}

// Entries of a thread where n (at most kBfsPer * T) of them are settled: thread t takes the entries
// from t * share on.
template <int T>
__device__ __forceinline__ int bfs_share(int32_t n) {
    return min((n + T - 1) / T, kBfsPer);
}

struct BfsArgs {
    const int32_t* __restrict__ queries;
    int64_t n_queries;
    int32_t k;
    int32_t n_nodes;
    const int64_t* __restrict__ inc_off;
    const int32_t* __restrict__ inc_q;
    const int32_t* __restrict__ start;   // [n_batches][n_start]
    int64_t n_batches;
    int32_t n_start;
    int32_t B1, B2;
    int32_t* __restrict__ vbar;          // [n_batches][B1]
    int32_t* __restrict__ batch;         // [n_batches][B2]
    int32_t* __restrict__ tuples;        // [n_batches][B2][k] or null
    int32_t* __restrict__ counts;        // [n_batches][2]
    uint32_t* tables;                    // per workgroup: query table, node table (unless in LDS)
    uint32_t slots_q, slots_v;           // powers of two
    uint32_t chunk;                      // candidates settled at a time: at most four per thread
    uint32_t most_new;                   // new queries looked at a time: those of a chunk, B2 at most
    uint32_t queue;                      // nodes a search can reach: entries of the queue in LDS
    uint32_t* err;
};

// Dynamic LDS of a workgroup, in 32-bit words: the lists of a chunk and, with kLds, the queue of
// nodes and both tables.
struct BfsLds {
    uint32_t new_q, node_slot, queue, tables, total;
};
__host__ __device__ inline BfsLds bfs_lds(uint32_t most_new, uint32_t queue, uint32_t slots, bool in_lds) {
    BfsLds o;
    o.new_q = 0;                           // newly reached queries, in order
    o.node_slot = o.new_q + most_new;      // slots of their nodes
    o.queue = (o.node_slot + most_new * kBfsMaxK + 3) / 4 * 4;
    o.tables = o.queue + (in_lds ? (queue + 3) / 4 * 4 : 0);
    o.total = o.tables + (in_lds ? 2 * slots : 0);
    return o;
}

// kPerSimd: waves of a SIMD that the registers leave room for.  Eight take more of the scalar ones out to
// lanes of vector ones, and are taken where LDS has room for as many searches: 2,048 of 128 queries 39 us,
// with four 45 (which are seven, as it comes out); 436 of 600 queries 62 and 60.
template <int T, bool kLds, int kPerSimd>
__global__ __launch_bounds__(T, kPerSimd) void bfs_batch_kernel(BfsArgs a) {
    __shared__ uint32_t wave_sums[T / kWave];
    __shared__ uint32_t pre[T + 1];              // candidates before each node of the stretch
    __shared__ int64_t list_at[T];               // where its list begins
    extern __shared__ __align__(16) uint32_t lds32[];
    const BfsLds lay = bfs_lds(a.most_new, a.queue, a.slots_q + a.slots_v, kLds);
    uint32_t* const new_q = lds32 + lay.new_q;
    uint32_t* const node_slot = lds32 + lay.node_slot;
    uint32_t* const queue = lds32 + lay.queue;   // kLds only

    const int tid = threadIdx.x;
    const int k = a.k;
    uint32_t* q_tab;
    if constexpr (kLds) {
        q_tab = lds32 + lay.tables;
    } else {
        q_tab = a.tables + (size_t)blockIdx.x * 2u * ((size_t)a.slots_q + a.slots_v);
    }
    uint32_t* v_tab = q_tab + 2u * (size_t)a.slots_q;
    const uint32_t q_mask = a.slots_q - 1u, v_mask = a.slots_v - 1u;
    const int64_t n_entries = a.n_queries * k;
    bool bad_id = false, bad_lists = false, table_full = false;

    for (int64_t b = blockIdx.x; b < a.n_batches; b += gridDim.x) {
        int32_t* vbar = a.vbar + b * a.B1;
        int32_t* batch = a.batch + b * a.B2;
        int32_t* tuples = a.tuples ? a.tuples + b * (int64_t)a.B2 * k : nullptr;
        const int32_t* start = a.start + b * (int64_t)a.n_start;

        // both tables empty (they lie back to back; 16 bytes a store)
        uint4* clear = reinterpret_cast<uint4*>(q_tab);
        for (uint32_t i = tid; i < (a.slots_q + a.slots_v) / 2u; i += T)
            clear[i] = make_uint4(kBfsEmpty, kBfsEmpty, kBfsEmpty, kBfsEmpty);
        if constexpr (!kLds) __threadfence();
        __syncthreads();

        uint32_t n_v = 0, n_b = 0;
        // the seed-set: distinct start nodes in the order given, B1 at most
        for (int32_t s0 = 0; s0 < a.n_start && n_v < (uint32_t)a.B1; s0 += T * kBfsPer) {
            const int32_t per = bfs_share<T>(a.n_start - s0);
            const int32_t s1 = min(a.n_start, s0 + per * T);
            uint32_t slot[kBfsPer];
            int32_t node[kBfsPer];
#pragma unroll
            for (int r = 0; r < kBfsPer; ++r) {
                const int32_t i = s0 + tid * per + r;
                slot[r] = kBfsEmpty;
                node[r] = -1;
                if (r < per && i < s1) {
                    node[r] = start[i];
                    if ((uint32_t)node[r] < (uint32_t)a.n_nodes) {
                        slot[r] = insert_min(v_tab, v_mask, (uint32_t)node[r], (uint32_t)i);
                        table_full |= slot[r] == kBfsEmpty;
                    } else {
                        bad_id = true;
                    }
                }
            }
            __syncthreads();
            uint32_t own = 0;
#pragma unroll
            for (int r = 0; r < kBfsPer; ++r) {
                const int32_t i = s0 + tid * per + r;
                const bool mine = slot[r] != kBfsEmpty && table_load<kLds>(&v_tab[2 * slot[r] + 1]) == (uint32_t)i;
                own |= mine ? 1u << r : 0u;
            }
            uint32_t total;
            uint32_t at = n_v + bfs_block_scan<T>((uint32_t)__popc(own), &total, wave_sums);
#pragma unroll
            for (int r = 0; r < kBfsPer; ++r)
                if (own & (1u << r)) {
                    if (at < (uint32_t)a.B1) {
                        vbar[at] = node[r];
                        if constexpr (kLds) queue[at] = (uint32_t)node[r];
                    }
                    at += 1;
                }
            n_v = min(n_v + total, (uint32_t)a.B1);
            __syncthreads();
        }

        bool done = n_v == (uint32_t)a.B1;
        uint32_t head = 0;       // next node of the queue
        uint32_t j_cur = 0;      // entries of its query list already taken
        uint32_t cand_base = 0;  // candidates numbered so far
        while (!done && head < n_v) {
            // the stretch: nodes head .. head+nf, thread t looks at node head+t
            const uint32_t nf = min((uint32_t)T, n_v - head);
            uint32_t deg = 0;
            if ((uint32_t)tid < nf) {
                const int32_t u = kLds ? (int32_t)queue[head + tid] : vbar[head + tid];
                list_at[tid] = a.inc_off[u];
                const int64_t len = a.inc_off[u + 1] - list_at[tid] - (tid == 0 ? (int64_t)j_cur : 0);
                bad_lists |= len < 0;
                // a list longer than a chunk is taken in pieces; how much longer does not matter
                deg = (uint32_t)max((int64_t)0, min(len, (int64_t)a.chunk + 1));
            }
            uint32_t total;
            const uint32_t excl = bfs_block_scan<T>(deg, &total, wave_sums);
            pre[tid] = excl;
            if (tid == T - 1) pre[T] = total;
            // nodes taken whole: the longest prefix of the stretch with at most a.chunk entries
            const bool whole = (uint32_t)tid < nf && excl + deg <= a.chunk;
            uint32_t take;
            if constexpr (T == kWave) {
                __syncthreads();
                take = (uint32_t)__popcll(__ballot(whole));
            } else {
                take = (uint32_t)__syncthreads_count(whole);
            }
            const bool partial = take == 0;  // the first node's list alone is longer than a chunk
            const uint32_t n_c = partial ? a.chunk : pre[take];
            const uint32_t n_src = partial ? 1u : take;
            const int per_c = bfs_share<T>((int32_t)n_c);

            // candidates: entry j of node t' of the stretch, numbered cand_base + c
            uint32_t cand_q[kBfsPer], cand_slot[kBfsPer];  // query of each, and its slot in the query table
#pragma unroll
            for (int r = 0; r < kBfsPer; ++r) {
                const uint32_t c = (uint32_t)(tid * per_c + r);
                cand_q[r] = 0u;
                cand_slot[r] = kBfsEmpty;
                if (r < per_c && c < n_c) {
                    uint32_t lo = 0, hi = n_src;  // last node with pre[node] <= c
                    while (hi - lo > 1) {
                        const uint32_t mid = (lo + hi) >> 1;
                        if (pre[mid] <= c) {
                            lo = mid;
                        } else {
                            hi = mid;
                        }
                    }
                    const int64_t e = list_at[lo] + (lo == 0 ? (int64_t)j_cur : 0) + (c - pre[lo]);
                    if (e >= 0 && e < n_entries) cand_q[r] = (uint32_t)a.inc_q[e];
                    if (e >= 0 && e < n_entries && (int64_t)cand_q[r] < a.n_queries) {
                        cand_slot[r] = insert_min(q_tab, q_mask, cand_q[r], cand_base + c);
                        table_full |= cand_slot[r] == kBfsEmpty;
                    } else {
                        bad_lists = true;
                    }
                }
            }
            __syncthreads();
            // the candidates that kept their query, in order: the newly reached queries
            uint32_t own = 0;
#pragma unroll
            for (int r = 0; r < kBfsPer; ++r) {
                const uint32_t c = (uint32_t)(tid * per_c + r);
                if (cand_slot[r] != kBfsEmpty && table_load<kLds>(&q_tab[2 * cand_slot[r] + 1]) == cand_base + c)
                    own |= 1u << r;
            }
            uint32_t n_new;
            uint32_t at = bfs_block_scan<T>((uint32_t)__popc(own), &n_new, wave_sums);
            // no more of them can be taken than the batch has room for
            const uint32_t n_look = min(n_new, (uint32_t)a.B2 - n_b);
            const int per_q = bfs_share<T>((int32_t)n_look);
#pragma unroll
            for (int r = 0; r < kBfsPer; ++r)
                if (own & (1u << r)) {
                    const uint32_t q = cand_q[r];
                    if (at < n_look) {
                        new_q[at] = q;
                    } else {  // B2 queries come before it: only its node ids are checked
                        for (int j = 0; j < k; ++j)
                            bad_id |= (uint32_t)a.queries[(int64_t)q * k + j] >= (uint32_t)a.n_nodes;
                    }
                    at += 1;
                }
            __syncthreads();

            // their nodes: node (i, j) is numbered n_start + (n_b + i) * k + j
            int32_t nodes[kBfsPer][kBfsMaxK];
#pragma unroll
            for (int r = 0; r < kBfsPer; ++r) {
                const uint32_t i = (uint32_t)(tid * per_q + r);
                if (r < per_q && i < n_look) {
                    const int64_t q = new_q[i];
#pragma unroll
                    for (int j = 0; j < kBfsMaxK; ++j) nodes[r][j] = j < k ? a.queries[q * k + j] : 0;
#pragma unroll
                    for (int j = 0; j < kBfsMaxK; ++j) {
                        if (j >= k) break;
                        const int32_t x = nodes[r][j];
                        uint32_t slot = kBfsEmpty;
                        if ((uint32_t)x < (uint32_t)a.n_nodes) {
                            slot = insert_min(v_tab, v_mask, (uint32_t)x,
                                              (uint32_t)a.n_start + (n_b + i) * (uint32_t)k + (uint32_t)j);
                            table_full |= slot == kBfsEmpty;
                        } else {
                            bad_id = true;
                        }
                        node_slot[i * kBfsMaxK + j] = slot;
                    }
                }
            }
            __syncthreads();
            uint32_t fresh[kBfsPer];  // bit j: node j of the query is new and first named here
            uint32_t n_fresh = 0;
#pragma unroll
            for (int r = 0; r < kBfsPer; ++r) {
                const uint32_t i = (uint32_t)(tid * per_q + r);
                fresh[r] = 0;
                if (r < per_q && i < n_look) {
                    for (int j = 0; j < k; ++j) {
                        const uint32_t slot = node_slot[i * kBfsMaxK + j];
                        if (slot != kBfsEmpty &&
                            table_load<kLds>(&v_tab[2 * slot + 1]) ==
                                (uint32_t)a.n_start + (n_b + i) * (uint32_t)k + (uint32_t)j)
                            fresh[r] |= 1u << j;
                    }
                    n_fresh += (uint32_t)__popc(fresh[r]);
                }
            }
            uint32_t all_fresh;
            uint32_t before = n_v + bfs_block_scan<T>(n_fresh, &all_fresh, wave_sums);
            // a query is taken if the queue would have reached it: room for its nodes, and neither
            // limit met by the queries before it
            uint32_t n_ok = 0, nodes_ok = 0;
            uint32_t first_at[kBfsPer];
#pragma unroll
            for (int r = 0; r < kBfsPer; ++r) {
                const uint32_t i = (uint32_t)(tid * per_q + r);
                const uint32_t mine = (uint32_t)__popc(fresh[r]);
                first_at[r] = before;
                const bool ok = r < per_q && i < n_look && before < (uint32_t)a.B1 &&
                                before + mine <= (uint32_t)a.B1;
                if (ok) {
                    n_ok += 1;
                    nodes_ok += mine;
                } else {
                    fresh[r] = 0xFFFFFFFFu;  // not taken
                }
                before += mine;
            }
            // (at most kBfsMaxChunk queries of three nodes: both sums in one word)
            static_assert(kBfsMaxChunk * kBfsMaxK < 1 << 16, "halves of a word");
            uint32_t both;
            (void)bfs_block_scan<T>(nodes_ok << 16 | n_ok, &both, wave_sums);
            const uint32_t took = both & 0xFFFFu, took_nodes = both >> 16;
#pragma unroll
            for (int r = 0; r < kBfsPer; ++r) {
                const uint32_t i = (uint32_t)(tid * per_q + r);
                if (fresh[r] != 0xFFFFFFFFu) {
                    const int64_t q = new_q[i];
                    batch[n_b + i] = (int32_t)q;
                    uint32_t at_v = first_at[r];
#pragma unroll
                    for (int j = 0; j < kBfsMaxK; ++j) {
                        if (j >= k) break;
                        const int32_t x = nodes[r][j];
                        if (tuples) tuples[(int64_t)(n_b + i) * k + j] = x;
                        if (fresh[r] & (1u << j)) {
                            vbar[at_v] = x;
                            if constexpr (kLds) queue[at_v] = (uint32_t)x;
                            at_v += 1;
                        }
                    }
                }
            }
            n_b += took;
            n_v += took_nodes;
            cand_base += n_c;
            if (partial) {
                j_cur += n_c;
            } else {
                head += take;
                j_cur = 0;
            }
            done = took < n_new || n_b == (uint32_t)a.B2 || n_v == (uint32_t)a.B1;
            __syncthreads();  // vbar and the LDS lists are complete before the next stretch
        }
        if (tid == 0) {
            a.counts[2 * b] = (int32_t)n_v;
            a.counts[2 * b + 1] = (int32_t)n_b;
        }
        __syncthreads();
    }
    raise_error(a.err, bad_id, kDevBadQuery);
    raise_error(a.err, bad_lists, kDevBadTable);
    raise_error(a.err, table_full, kDevStall);
}

uint32_t pow2_at_least(uint64_t x) {
    uint32_t p = 1;
    while (p < x) p <<= 1;
    return p;
}

}  // namespace

// Candidates settled at a time: every one of them is entered into the query table before the limits
// cut, so small batches take small bites.
static uint32_t bfs_chunk(int32_t B2) {
    const uint32_t want = pow2_at_least(4ull * (uint64_t)B2);
    return want < 64u ? 64u : (want > (uint32_t)kBfsMaxChunk ? (uint32_t)kBfsMaxChunk : want);
}
// One wavefront per search where a chunk fits its four candidates a lane: more searches in
// flight per compute unit, and their barriers cost nothing.
static int bfs_threads(int32_t B2) { return bfs_chunk(B2) <= (uint32_t)(kWave * kBfsPer) ? kWave : kBfsMaxThreads; }

// Nodes a search can reach: its start nodes and those of B2 queries, B1 at most.
static uint64_t bfs_nodes(int32_t n_start, int32_t B1, int32_t B2, int32_t k) {
    const uint64_t reach = (uint64_t)n_start + (uint64_t)B2 * (uint64_t)k;
    return reach < (uint64_t)B1 ? reach : (uint64_t)B1;
}
// Slots of the two hash tables of one workgroup: at most half of them are ever used (in LDS, where
// a probe costs little and room is short, four fifths).  Besides the queries and nodes of the batch
// and the start nodes, the candidates of one chunk and their nodes get in.
struct BfsTables {
    uint32_t slots_q, slots_v;
    size_t bytes() const { return 2u * sizeof(uint32_t) * ((size_t)slots_q + slots_v); }
};
static BfsTables bfs_tables(int32_t n_start, int32_t B1, int32_t B2, int32_t k, bool in_lds) {
    const uint64_t q = (uint64_t)B2 + bfs_chunk(B2);
    const uint64_t v = (uint64_t)n_start + (uint64_t)B2 * (uint64_t)k;
    if (in_lds) return BfsTables{pow2_at_least(q + q / 4), pow2_at_least(v + v / 4)};
    return BfsTables{pow2_at_least(2 * q), pow2_at_least(2 * v)};
}
static uint32_t bfs_most_new(int32_t B2) {
    return (uint32_t)B2 < bfs_chunk(B2) ? (uint32_t)B2 : bfs_chunk(B2);
}
static size_t bfs_lds_bytes(int32_t n_start, int32_t B1, int32_t B2, int32_t k, bool in_lds) {
    const BfsTables t = bfs_tables(n_start, B1, B2, k, in_lds);
    return sizeof(uint32_t) * (size_t)bfs_lds(bfs_most_new(B2), (uint32_t)bfs_nodes(n_start, B1, B2, k),
                                              t.slots_q + t.slots_v, in_lds).total;
}
static bool bfs_in_lds(int32_t n_start, int32_t B1, int32_t B2, int32_t k) {
    // (the sizes first: the words of large tables need not fit 32 bits)
    const size_t most = bfs_threads(B2) == kWave ? kBfsLdsMost : kBfsLdsMostWide;
    return bfs_tables(n_start, B1, B2, k, true).bytes() <= most &&
           bfs_lds_bytes(n_start, B1, B2, k, true) <= most;
}

// Searches in flight with tables in global memory: 16 waves a compute unit, fewer if their tables
// would pass 4 GiB.
static int bfs_grid(int n_cu, int64_t n_batches, size_t table_bytes, int threads) {
    int64_t resident = (int64_t)n_cu * (16 * kWave / threads);
    const int64_t by_memory = (int64_t)(((size_t)4 << 30) / table_bytes);
    if (resident > by_memory) resident = by_memory > 0 ? by_memory : 1;
    return (int)(n_batches < resident ? n_batches : resident);
}

size_t bfs_scratch_bytes(int n_cu, int64_t n_batches, int32_t n_start, int32_t B1, int32_t B2,
                         int32_t k) {
    if (bfs_in_lds(n_start, B1, B2, k)) return 0;
    const size_t per = bfs_tables(n_start, B1, B2, k, false).bytes();
    return (size_t)bfs_grid(n_cu, n_batches, per, bfs_threads(B2)) * per;
}

template <int T, bool kLds, int kPerSimd>
static hipError_t launch_bfs_cfg(hipStream_t stream, int64_t grid, size_t lds_bytes, const BfsArgs& a) {
    if (lds_bytes > 48 * 1024) {
        hipError_t rc = hipFuncSetAttribute(reinterpret_cast<const void*>(bfs_batch_kernel<T, kLds, kPerSimd>),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (rc != hipSuccess) return rc;
    }
    hipLaunchKernelGGL((bfs_batch_kernel<T, kLds, kPerSimd>), dim3((unsigned)grid), dim3(T), lds_bytes, stream, a);
    return hipGetLastError();
}

hipError_t launch_bfs_batches(hipStream_t stream, int n_cu, const int32_t* queries,
                              int64_t n_queries, int32_t k, int32_t n_nodes, const int64_t* inc_off,
                              const int32_t* inc_q, const int32_t* start, int64_t n_batches,
                              int32_t n_start, int32_t B1, int32_t B2, int32_t* vbar, int32_t* batch,
                              int32_t* tuples, int32_t* counts, void* scratch, uint32_t* err) {
    if (n_batches == 0) return hipSuccess;
    BfsArgs a;
    a.queries = queries;
    a.n_queries = n_queries;
    a.k = k;
    a.n_nodes = n_nodes;
    a.inc_off = inc_off;
    a.inc_q = inc_q;
    a.start = start;
    a.n_batches = n_batches;
    a.n_start = n_start;
    a.B1 = B1;
    a.B2 = B2;
    a.vbar = vbar;
    a.batch = batch;
    a.tuples = tuples;
    a.counts = counts;
    a.tables = static_cast<uint32_t*>(scratch);
    const bool in_lds = bfs_in_lds(n_start, B1, B2, k);
    const BfsTables tables = bfs_tables(n_start, B1, B2, k, in_lds);
    a.slots_q = tables.slots_q;
    a.slots_v = tables.slots_v;
    a.chunk = bfs_chunk(B2);
    a.most_new = bfs_most_new(B2);
    a.queue = in_lds ? (uint32_t)bfs_nodes(n_start, B1, B2, k) : 0u;
    a.err = err;
    const int threads = bfs_threads(B2);
    const size_t lds_bytes = bfs_lds_bytes(n_start, B1, B2, k, in_lds);
    if (in_lds) {  // a workgroup per search, the hardware hands them out
        const int64_t grid = n_batches < 0x7FFFFF ? n_batches : 0x7FFFFF;
        if (threads == kWave) return launch_bfs_cfg<kWave, true, 8>(stream, grid, lds_bytes, a);
        if (lds_bytes <= kBfsLdsEight) return launch_bfs_cfg<kBfsMaxThreads, true, 8>(stream, grid, lds_bytes, a);
        return launch_bfs_cfg<kBfsMaxThreads, true, 4>(stream, grid, lds_bytes, a);
    }
    const int grid = bfs_grid(n_cu, n_batches, tables.bytes(), threads);
    if (threads == kWave) return launch_bfs_cfg<kWave, false, 4>(stream, grid, lds_bytes, a);
    return launch_bfs_cfg<kBfsMaxThreads, false, 4>(stream, grid, lds_bytes, a);
}

}  // namespace surel
