// Query-based subgraph joining in its set-union form (Sec. 3.4): for a query tuple
// (b_1..b_K) the ascending union of the K node sets, and per union node the K count
// vectors in tuple order, zeros where the node is absent from a set.  How a query's lists are
// united and its rows written: join_core.h.
//
// Long query lists take two launches.  Counting: every query's union rows (an exclusive scan then
// turns the counts into join_off).  Filling: join_off is given (by that scan, or kept by the
// caller from an earlier call), the rows are written.  A wavefront handles one query at a time;
// the K sorted id lists are staged in LDS.  (Doing both in one launch, with the offsets from a
// scanner wave inside the kernel as the fused walk + RPE kernel has them, was built and measured:
// a wave has to wait for its query's offset between uniting and writing, which took 10.0 ms
// against 0.83 + 5.6 ms for the two launches on the 2.9M-node workload; holding one query back to
// hide that wait doubles the LDS a wave needs, and the filling launch with that footprint alone
// takes 8.9 ms.)
//
// Short query lists (join_small_kernel) take one launch of one workgroup per query, as many as the
// device has room for at a time: there a launch's time is the chain of one query, so several
// wavefronts share a query, and the offsets come from the words that the workgroups publish
// (small_scan.h).
#include "device_util.h"
#include "join_core.h"
#include "kernels.h"
#include "small_scan.h"

namespace surel {

// Filling.  One wavefront per workgroup and one query per wavefront; the grid covers the query
// list.  The hardware hands workgroups out as others retire, which keeps every compute unit
// full whatever the queries' sizes are and however many waves it really holds.  (A grid of
// exactly as many waves as the occupancy query promises, each looping over a strided share of
// the queries, was slower: where the device held fewer workgroups than promised, the surplus
// ran as a tail after the others, +25 % on one workload; and with four waves to a workgroup a
// slot stays taken until the slowest of the four is done.)
// join_off is complete (the caller's, or the scan of a counting launch).  A query whose union
// does not have the join_off[q+1] - join_off[q] rows that the offsets give it is flagged and
// writes nothing.
template <int K, int LT>
__global__ __launch_bounds__(kWave) void join_fill_kernel(
    const int64_t* __restrict__ rpe_off, const int32_t* __restrict__ rpe_ids,
    const uint16_t* __restrict__ rpe_cnt, int64_t n_blocks, int32_t max_set,
    const int32_t* __restrict__ queries, int64_t n_queries,
    const int64_t* __restrict__ join_off, int64_t cap_rows, int32_t* __restrict__ out_ids,
    uint16_t* __restrict__ out_cnt, int first_place, uint16_t absent16, uint32_t* __restrict__ err) {
    extern __shared__ __align__(16) uint32_t base[];
    const JoinTeam<false> team{lane_id(), 0, 1, nullptr};
    const int lane = team.lane;
    const JoinLds lay = join_lds_layout(K, max_set, LT, 1);
    // (written as a loop over the wave's one query: the compiler's code for this form makes the
    // launch 2 % faster on the 2.9M-node workload than the same statements in a row)
    constexpr int kPerWave = 1;
    const int64_t q_first = (int64_t)blockIdx.x * kPerWave;
#pragma unroll 1
    for (int64_t q = q_first; q < min(q_first + kPerWave, n_queries); ++q) {
        JoinQuery<K> jq;
        const uint32_t problem = join_lookup<K>(q, rpe_off, n_blocks, max_set, queries, jq);
        const int64_t off = join_off[q];
        const bool past = join_off[n_queries] * (int64_t)(4 + 2 * K * LT) > kPastBytes;
        const int first_bit = past ? (int)((off + first_place) & (kRowsAlign - 1)) : 0;
        int rows = 0;  // an unusable query yields no rows
        if (problem != 0) {
            if (lane == 0) atomicOr(err, problem);
        } else {
            // the same in every lane; said so, the loops over the rows are scalar loops
            rows = __builtin_amdgcn_readfirstlane(join_unite<K, false>(
                base, lay, max_set, jq, team, first_bit, [&](uint32_t* dst, int j) {
                    stage_words<8>(dst, reinterpret_cast<const uint32_t*>(rpe_ids + jq.lo[j]),
                                   jq.n[j], lane);
                }));
            if constexpr (K == 3) jq.n01 = __builtin_amdgcn_readfirstlane(jq.n01);
            wave_sync();
        }
        if (join_off[q + 1] - off != (int64_t)rows) {
            if (lane == 0) atomicOr(err, kDevBadSizes);
        } else if (rows > 0 && off + rows > cap_rows) {
            if (lane == 0) atomicOr(err, kDevCapacity);
        } else if (rows > 0) {
            if (past)
                join_write<K, LT, false, true>(base, lay, jq, first_bit, rows, off, rpe_cnt, max_set,
                                               out_ids, out_cnt, absent16, team);
            else
                join_write<K, LT, false, false>(base, lay, jq, 0, rows, off, rpe_cnt, max_set, out_ids,
                                                out_cnt, absent16, team);
        }
        wave_sync();
    }
}

// Union rows of query q, for a workgroup that helps another one (one wavefront, no LDS): the nodes
// of a list that none of the lists before it holds, by bisection.  (Of lists that are not ascending,
// which no table has, it may count other rows than the merge; nothing is written past cap_rows.)
template <int K>
__device__ __forceinline__ uint32_t join_small_rows(int q, const int64_t* __restrict__ rpe_off,
                                                    const int32_t* __restrict__ rpe_ids,
                                                    int64_t n_blocks, int32_t max_set,
                                                    const int32_t* __restrict__ queries, int lane) {
    JoinQuery<K> jq;
    if (join_lookup<K>(q, rpe_off, n_blocks, max_set, queries, jq) != 0) return 0;
    uint32_t rows = 0;
#pragma unroll
    for (int j = 0; j < K; ++j) {
#pragma unroll 1
        for (int t = lane; t < jq.n[j]; t += kWave) {
            const int32_t x = rpe_ids[jq.lo[j] + t];
            bool known = false;
#pragma unroll
            for (int i = 0; i < j; ++i) {
                int lo = 0, hi = jq.n[i];
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (rpe_ids[jq.lo[i] + mid] < x) {
                        lo = mid + 1;
                    } else {
                        hi = mid;
                    }
                }
                known = known || (lo < jq.n[i] && rpe_ids[jq.lo[i] + lo] == x);
            }
            rows += known ? 0u : 1u;
        }
    }
    return wave_bcast_u32(wave_incl_sum(rows), kWave - 1);
}

// One workgroup of n_waves wavefronts per query (see the file's head).  out_ids null: only the
// offsets are wanted.  h_total (optional): host memory that gets the row total as well.
// What bounds it: the chain of one query, about six trips to memory and the merge (10.8 us for 32
// pairs of M = 200, m = 4).  A call that reports its total, against the counting launch, the three
// launches of the scan, the filling launch and the copy of the total: 25 instead of 76 us for 32
// such pairs, 32 instead of 86 for 1,000, 57 instead of 101 for 4,096.
template <int K, int LT>
__global__ __launch_bounds__(1024) void join_small_kernel(
    const int64_t* __restrict__ rpe_off, const int32_t* __restrict__ rpe_ids,
    const uint16_t* __restrict__ rpe_cnt, int64_t n_blocks, int32_t max_set,
    const int32_t* __restrict__ queries, int32_t n_queries, int64_t* __restrict__ join_off,
    int64_t cap_rows, int32_t* __restrict__ out_ids, uint16_t* __restrict__ out_cnt,
    uint16_t absent16, SmallScan* __restrict__ ss, uint32_t spin_limit, int64_t* h_total,
    uint32_t* __restrict__ err) {
    extern __shared__ __align__(16) uint32_t base[];
    __shared__ uint32_t sums[1024 / kWave];
    __shared__ int64_t s_off;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const JoinTeam<true> team{lane_id(), wave, (int)(blockDim.x >> 6), sums};
    const int lane = team.lane;
    const JoinLds lay = join_lds_layout(K, max_set, LT, team.n_waves);
    const int q = (int)blockIdx.x;
    uint32_t tag = 0;
    if (wave == 0) tag = small_scan_tag(ss);
    JoinQuery<K> jq;
    const uint32_t problem = join_lookup<K>(q, rpe_off, n_blocks, max_set, queries, jq);
    int rows = 0;  // an unusable query yields no rows
    if (problem != 0) {
        if (threadIdx.x == 0) atomicOr(err, problem);
    } else {
        rows = __builtin_amdgcn_readfirstlane(join_unite<K, true>(
            base, lay, max_set, jq, team, 0, [&](uint32_t* dst, int j) {
                const uint32_t* src = reinterpret_cast<const uint32_t*>(rpe_ids + jq.lo[j]);
                stage_words<4>(dst, src, jq.n[j], team.tid(), team.threads());
            }));
        if constexpr (K == 3) jq.n01 = __builtin_amdgcn_readfirstlane(jq.n01);
    }
    if (wave == 0) {
        if (lane == 0) small_scan_publish(ss, q, tag, (uint32_t)rows);
        const int64_t before = small_scan_before(ss, q, tag, spin_limit, lane, [&](int j) {
            return join_small_rows<K>(j, rpe_off, rpe_ids, n_blocks, max_set, queries, lane);
        });
        if (lane == 0) {
            small_scan_done(ss, q, tag, n_queries);
            s_off = before;
            join_off[q] = before;
            if (q == n_queries - 1) {
                join_off[n_queries] = before + rows;
                if (h_total) *h_total = before + rows;
            }
        }
    }
    __syncthreads();
    const int64_t off = s_off;
    if (out_ids == nullptr || rows == 0) return;
    if (off + rows > cap_rows) {
        if (threadIdx.x == 0) atomicOr(err, kDevCapacity);
        return;
    }
    join_write<K, LT, true, false>(base, lay, jq, 0, rows, off, rpe_cnt, max_set, out_ids, out_cnt, absent16,
                            team);
}

// Counting.  A wavefront takes up to kCountQueries consecutive queries.  Their
// blocks are looked up by one lane each (block numbers, then the blocks' offsets: two round
// trips to memory for all of them), and while one query is counted in LDS the lists of the next one
// are already on their way into registers.
//
// Nothing is merged: the union has the rows of all lists less those of nodes that an earlier list
// holds.  A list's nodes set their bits in a hashed bit map; of the next list's nodes only those that
// find their bit set are put on a list and looked up in the earlier ones by bisection, 64 at a time:
// true repetitions and false ones, as many of a list as the map has bits set (276 ids in 8,192 bits 3.3
// in a hundred, 561 6.4; triples of 181 2.2 of the second list, 4.3 of the third).
// What bounds it: the lists' way from memory.  1,048,576 pairs of the 2.9M-node graph move 6.2 TB/s
// (23.7 M lines of 128 bytes, a tenth of them for the blocks' offsets) with 222 vector instructions
// a pair; triples of 181 nodes a list the vector instructions (0.74 of the time).
// By merge path, where every lane bisects and then merges its share node after node, it took 446
// instructions a pair and 0.63 ms, now 0.49; 262,144 triples of m = 3 0.36 -> 0.21; 65,536 pairs of
// 561 nodes a list 0.105 -> 0.075.
// Queries to a wave, for long lists: 4 / 8 / 16 pairs take 0.52 / 0.50 / 0.58 ms, 4 / 8 triples 0.239 /
// 0.234.  For shorter lists as few as leave 16 waves a compute unit: 4,694 triples of 500 nodes a list
// 33 us (eight to a wave 106), 20,000 pairs of 290 nodes 17 (23 where eight waves were enough).
constexpr int kCountQueries = 8;  // at most; fewer where the waves would not fill the device
constexpr int kCountStage = 8;  // words of a list a lane holds for the next query (512 ids)

// LDS of a counting wave, in 32-bit words: the bit map, the lists that are looked up in, and the
// nodes that wait for their look-up.
struct CountLds {
    int map_bits;  // log2 of the words of the bit map: max_set ids set one bit in eight at most (the
                   // third list of a triple finds two lists' bits, one in four at most)
    int lists, waiting;
    int total;
};
__host__ __device__ constexpr CountLds count_lds_layout(int K, int max_set) {
    CountLds o{};
    o.map_bits = 8;  // cleared 16 bytes a lane
    while ((4 << o.map_bits) < max_set) o.map_bits += 1;
    o.lists = 1 << o.map_bits;
    o.waiting = o.lists + (K - 1) * max_set;
    o.total = o.waiting + max_set;
    return o;
}

// Whether the ascending list[0 .. n) holds x; steps: 2^steps > n.
__device__ __forceinline__ bool list_holds(const uint32_t* list, int n, int steps, uint32_t x) {
    int below = 0;  // ids of the list that are known to be smaller than x
    for (int half = 1 << (steps - 1); half > 0; half >>= 1) {
        const int at = below + half;
        if (at <= n && list[at - 1] < x) below = at;
    }
    return below < n && list[below] == x;
}

template <int K>
__global__ __launch_bounds__(kWave) void join_count_kernel(
    const int64_t* __restrict__ rpe_off, const int32_t* __restrict__ rpe_ids, int64_t n_blocks,
    int32_t max_set, const int32_t* __restrict__ queries, int64_t n_queries,
    int per_wave, int32_t* __restrict__ counts, uint32_t* __restrict__ err) {
    extern __shared__ __align__(16) uint32_t base[];
    const CountLds lay = count_lds_layout(K, max_set);
    const int lane = lane_id();
    const int64_t q_first = (int64_t)blockIdx.x * per_wave;

    // lane l < kCountQueries looks up the blocks of query q_first + l
    int64_t my_lo[K];
    int my_n[K];
    uint32_t my_problem = 0;
#pragma unroll
    for (int j = 0; j < K; ++j) {
        my_lo[j] = 0;
        my_n[j] = 0;
    }
    if (lane < per_wave && q_first + lane < n_queries) {
        int32_t b[K];
#pragma unroll
        for (int j = 0; j < K; ++j) b[j] = queries[(q_first + lane) * K + j];
#pragma unroll
        for (int j = 0; j < K; ++j) {
            if (b[j] < 0 || (int64_t)b[j] >= n_blocks) {
                my_problem |= kDevBadQuery;
            } else {
                const int64_t a = rpe_off[b[j]];
                const int64_t len = rpe_off[b[j] + 1] - a;
                if (a < 0 || len < 0) {
                    my_problem |= kDevBadTable;
                } else if (len > (int64_t)max_set) {
                    my_problem |= kDevSetTooLarge;
                } else {
                    my_lo[j] = a;
                    my_n[j] = (int)len;
                }
            }
        }
        if (my_problem != 0) {  // the query is flagged and yields no rows
            atomicOr(err, my_problem);
#pragma unroll
            for (int j = 0; j < K; ++j) my_n[j] = 0;
        }
    }
    // query i's blocks, the same in every lane
    auto blocks_of = [&](int i, int64_t (&lo)[K], int (&n)[K]) {
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const uint32_t lo_l = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(uint64_t)my_lo[j], i);
            const uint32_t lo_h = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)my_lo[j] >> 32), i);
            lo[j] = (int64_t)(((uint64_t)lo_h << 32) | lo_l);
            n[j] = __builtin_amdgcn_readlane(my_n[j], i);
        }
    };
    // ids t0 .. t0 + 511 of a list, in the registers that it has ids for
    auto fetch = [&](uint32_t (&x)[kCountStage], int64_t lo, int t0, int n) {
        const int32_t* list = rpe_ids + lo;
#pragma unroll
        for (int u = 0; u < kCountStage; ++u) x[u] = any_value();
#pragma unroll
        for (int u = 0; u < kCountStage; ++u) {
            const int first = t0 + u * kWave;
            if (first >= n) break;
            x[u] = (uint32_t)list[(uint32_t)min(first + lane, n - 1)];
        }
    };
    // an id's bit in the map.  (The product of 24 bits takes a quarter of a full one's time; ids that
    // differ above them share a bit.)
    const uint32_t bit_shift = 27u - (uint32_t)lay.map_bits;
    auto bit_of = [&](uint32_t x) { return (uint32_t)__umul24(x, 0x9E3779u) >> bit_shift; };
    uint32_t* map = base;
    auto insert = [&](const uint32_t (&x)[kCountStage], int t0, int n, uint32_t* list) {
#pragma unroll
        for (int u = 0; u < kCountStage; ++u) {
            if (t0 + u * kWave >= n) break;
            const int t = t0 + u * kWave + lane;
            if (t < n) {
                const uint32_t b = bit_of(x[u]);
                list[t] = x[u];
                atomicOr(map + (b >> 5), 1u << (b & 31u));
            }
        }
    };
    uint32_t* waiting = base + lay.waiting;
    auto probe = [&](const uint32_t (&x)[kCountStage], int t0, int n, int& n_waiting) {
        // (registers that hold no ids read some word of the map, which is masked out)
        uint32_t word[kCountStage];
        const int n_words = n - t0;
#pragma unroll
        for (int h = 0; h < kCountStage; h += kCountStage / 2) {
            if (h * kWave >= n_words) break;
#pragma unroll
            for (int u = h; u < h + kCountStage / 2; ++u) word[u] = map[bit_of(x[u]) >> 5];
#pragma unroll
            for (int u = h; u < h + kCountStage / 2; ++u) {
                if (u * kWave >= n_words) break;
                const uint32_t set = (word[u] >> (bit_of(x[u]) & 31u)) & 1u;
                const uint64_t hits = __ballot(set != 0u) & __ballot(lane < n_words - u * kWave);
                if (hits != 0ull) {
                    const int rank = (int)__builtin_amdgcn_mbcnt_hi(
                        (uint32_t)(hits >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hits, 0u));
                    if (__builtin_amdgcn_inverse_ballot_w64(hits)) waiting[n_waiting + rank] = x[u];
                    n_waiting += __popcll(hits);
                }
            }
        }
    };
    const int steps = 32 - __builtin_clz((uint32_t)max_set);

    uint32_t staged[K][kCountStage];
    int64_t lo[K];
    int n[K];
    blocks_of(0, lo, n);
#pragma unroll
    for (int j = 0; j < K; ++j) fetch(staged[j], lo[j], 0, n[j]);
#pragma unroll 1
    for (int i = 0; i < per_wave; ++i) {
        const int64_t q = q_first + i;
        if (q >= n_queries) break;
        int64_t lo_now[K];
        int n_now[K];
#pragma unroll
        for (int j = 0; j < K; ++j) lo_now[j] = lo[j], n_now[j] = n[j];
        uint4* clear = reinterpret_cast<uint4*>(map);
        for (int t = lane; t < (1 << lay.map_bits) / 4; t += kWave) clear[t] = make_uint4(0u, 0u, 0u, 0u);
        wave_sync();
        int rows = n_now[0];
#pragma unroll
        for (int j = 0; j < K; ++j) {
            // the ids that the registers do not hold come from memory
            if (j > 0) {
                int n_waiting = 0;
                probe(staged[j], 0, n_now[j], n_waiting);
                for (int t0 = kCountStage * kWave; t0 < n_now[j]; t0 += kCountStage * kWave) {
                    uint32_t x[kCountStage];
                    fetch(x, lo_now[j], t0, n_now[j]);
                    probe(x, t0, n_now[j], n_waiting);
                }
                wave_sync();
                rows += n_now[j];
                for (int t0 = 0; t0 < n_waiting; t0 += kWave) {
                    const int t = t0 + lane;
                    const uint32_t x = waiting[min(t, n_waiting - 1)];
                    bool known = false;
#pragma unroll
                    for (int e = 0; e < j; ++e)
                        known = known || list_holds(base + lay.lists + e * max_set, n_now[e], steps, x);
                    rows -= __popcll(__ballot(known && t < n_waiting));
                }
            }
            if (j < K - 1) {
                uint32_t* list = base + lay.lists + j * max_set;
                insert(staged[j], 0, n_now[j], list);
                for (int t0 = kCountStage * kWave; t0 < n_now[j]; t0 += kCountStage * kWave) {
                    uint32_t x[kCountStage];
                    fetch(x, lo_now[j], t0, n_now[j]);
                    insert(x, t0, n_now[j], list);
                }
            } else if (i + 1 < per_wave && q + 1 < n_queries) {
                // the registers are free: the next query's lists
                blocks_of(i + 1, lo, n);
#pragma unroll
                for (int e = 0; e < K; ++e) fetch(staged[e], lo[e], 0, n[e]);
            }
            wave_sync();
        }
        if (lane == 0) counts[q] = rows;
    }
}

// What a launch is asked to do.
struct JoinJob {
    hipStream_t stream;
    int max_lds_bytes;
    const int64_t* rpe_off;
    const int32_t* rpe_ids;
    const uint16_t* rpe_cnt;
    int64_t n_blocks;
    int32_t m;
    int32_t max_set;
    const int32_t* queries;
    int64_t n_queries;
    int32_t* counts;          // counting launch: written
    const int64_t* join_off;  // filling launch: read
    int64_t cap_rows;
    int32_t* out_ids;
    uint16_t* out_cnt;
    uint16_t absent16;
    uint32_t* err;
    // the one-launch join
    int n_cu;
    int64_t* join_off_out;    // written
    SmallScan* small_scan;
    uint32_t spin_limit;
    int64_t* h_total;
    hipEvent_t done;
};

// Wavefronts of a query in the one-launch join: as many as the device has room for at four waves
// per SIMD (16 per compute unit), 16 at most.
static int join_small_waves(int64_t n_queries, int n_cu) {
    int w = 16;
    while (w > 1 && n_queries * w > (int64_t)n_cu * 16) w /= 2;
    return w;
}

static hipError_t allow_lds(const void* fn, size_t lds_bytes) {
    if (lds_bytes <= 48 * 1024) return hipSuccess;
    return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
}

template <int K, int LT>
static hipError_t launch_join_fill_cfg(const JoinJob& j) {
    const size_t lds_bytes = (size_t)join_lds_layout(K, j.max_set, LT, 1).total * 4;
    if (lds_bytes > (size_t)j.max_lds_bytes) return hipErrorInvalidValue;
    hipError_t rc = allow_lds(reinterpret_cast<const void*>(join_fill_kernel<K, LT>), lds_bytes);
    if (rc != hipSuccess) return rc;
    if (j.n_queries > 0x7FFFFFFFll) return hipErrorInvalidValue;
    const int first_place = join_first_place(j.out_ids, j.out_cnt, 2 * K * LT);
    hipLaunchKernelGGL((join_fill_kernel<K, LT>), dim3((unsigned)j.n_queries), dim3(kWave),
                       lds_bytes, j.stream, j.rpe_off, j.rpe_ids, j.rpe_cnt, j.n_blocks, j.max_set,
                       j.queries, j.n_queries, j.join_off, j.cap_rows, j.out_ids, j.out_cnt,
                       first_place, j.absent16, j.err);
    return hipGetLastError();
}

template <int K, int LT>
static hipError_t launch_join_small_cfg(const JoinJob& j) {
    const int W = join_small_waves(j.n_queries, j.n_cu);
    const size_t lds_bytes = (size_t)join_lds_layout(K, j.max_set, LT, W).total * 4;
    hipError_t rc = allow_lds(reinterpret_cast<const void*>(join_small_kernel<K, LT>), lds_bytes);
    if (rc != hipSuccess) return rc;
    launch_and_mark(join_small_kernel<K, LT>, dim3((unsigned)j.n_queries), dim3(W * kWave), lds_bytes,
                    j.stream, j.done, j.rpe_off, j.rpe_ids, j.rpe_cnt, j.n_blocks, j.max_set,
                    j.queries, (int32_t)j.n_queries, j.join_off_out, j.cap_rows, j.out_ids,
                    j.out_cnt, j.absent16, j.small_scan, j.spin_limit, j.h_total, j.err);
    return hipGetLastError();
}

// m + 1 at compile time
template <int K, bool kSmall>
static hipError_t launch_join_lt(const JoinJob& j) {
    switch (j.m + 1) {
#define SUREL_JOIN_LT(LT_) \
    case LT_: \
        if constexpr (kSmall) return launch_join_small_cfg<K, LT_>(j); \
        else return launch_join_fill_cfg<K, LT_>(j);
        SUREL_JOIN_LT(2)
        SUREL_JOIN_LT(3)
        SUREL_JOIN_LT(4)
        SUREL_JOIN_LT(5)
        SUREL_JOIN_LT(6)
        SUREL_JOIN_LT(7)
        SUREL_JOIN_LT(8)
        SUREL_JOIN_LT(9)
        SUREL_JOIN_LT(10)
        SUREL_JOIN_LT(11)
        SUREL_JOIN_LT(12)
        SUREL_JOIN_LT(13)
        SUREL_JOIN_LT(14)
        SUREL_JOIN_LT(15)
        SUREL_JOIN_LT(16)
#undef SUREL_JOIN_LT
        default: return hipErrorInvalidValue;
    }
}

template <int K>
static hipError_t launch_join_count_k(const JoinJob& j) {
    const size_t lds_bytes = (size_t)count_lds_layout(K, j.max_set).total * 4;
    if (lds_bytes > (size_t)j.max_lds_bytes) return hipErrorInvalidValue;
    hipError_t rc = allow_lds(reinterpret_cast<const void*>(join_count_kernel<K>), lds_bytes);
    if (rc != hipSuccess) return rc;
    int per_wave = (int)(j.n_queries / ((int64_t)j.n_cu * 16));
    per_wave = per_wave < 1 ? 1 : per_wave > kCountQueries ? kCountQueries : per_wave;
    const int64_t blocks = (j.n_queries + per_wave - 1) / per_wave;
    hipLaunchKernelGGL((join_count_kernel<K>), dim3((unsigned)blocks), dim3(kWave), lds_bytes,
                       j.stream, j.rpe_off, j.rpe_ids, j.n_blocks, j.max_set, j.queries,
                       j.n_queries, per_wave, j.counts, j.err);
    return hipGetLastError();
}

hipError_t launch_join_count(hipStream_t stream, int max_lds_bytes, int n_cu, const int64_t* rpe_off,
                             const int32_t* rpe_ids, int64_t n_blocks, int32_t max_set,
                             const int32_t* queries, int64_t n_queries, int32_t k, int32_t* counts,
                             uint32_t* err) {
    JoinJob j{};
    j.stream = stream, j.max_lds_bytes = max_lds_bytes, j.n_cu = n_cu;
    j.rpe_off = rpe_off, j.rpe_ids = rpe_ids, j.n_blocks = n_blocks, j.m = 1, j.max_set = max_set;
    j.queries = queries, j.n_queries = n_queries, j.counts = counts, j.err = err;
    if (n_queries == 0) return hipSuccess;
    if (k == 2) return launch_join_count_k<2>(j);
    if (k == 3) return launch_join_count_k<3>(j);
    return hipErrorInvalidValue;
}

hipError_t launch_join_fill(hipStream_t stream, int max_lds_bytes, const int64_t* rpe_off,
                            const int32_t* rpe_ids, const uint16_t* rpe_cnt, int64_t n_blocks,
                            int32_t m, int32_t max_set, const int32_t* queries, int64_t n_queries,
                            int32_t k, const int64_t* join_off, int64_t cap_rows, int32_t* out_ids,
                            uint16_t* out_cnt, uint16_t absent16, uint32_t* err) {
    JoinJob j{};
    j.stream = stream, j.max_lds_bytes = max_lds_bytes;
    j.rpe_off = rpe_off, j.rpe_ids = rpe_ids, j.rpe_cnt = rpe_cnt, j.n_blocks = n_blocks, j.m = m;
    j.max_set = max_set, j.queries = queries, j.n_queries = n_queries, j.join_off = join_off;
    j.cap_rows = cap_rows, j.out_ids = out_ids, j.out_cnt = out_cnt, j.absent16 = absent16;
    j.err = err;
    if (n_queries == 0) return hipSuccess;
    if (k == 2) return launch_join_lt<2, false>(j);
    if (k == 3) return launch_join_lt<3, false>(j);
    return hipErrorInvalidValue;
}

// The one-launch join (up to 4,096 queries on 256 compute units; at that size it still takes half
// the time of the separate launches) is for query lists whose workgroups the device can hold all at
// once, so that hardly one waits for another to start: four waves per SIMD (its 88 registers leave
// room for five) and 160 KB of LDS per compute unit.
bool join_is_small(int n_cu, int max_lds_bytes, int32_t max_set, int32_t m, int64_t n_queries,
                   int32_t k) {
    if (n_queries < 1 || n_queries > kSmallScanMax) return false;
    const int w = join_small_waves(n_queries, n_cu);
    if (n_queries * w > (int64_t)n_cu * 16) return false;
    const int64_t lds = (int64_t)join_lds_layout(k, max_set, m + 1, w).total * 4 + 256;
    if (lds > max_lds_bytes) return false;
    const int64_t per_cu = 160 * 1024 / lds;
    return n_queries <= per_cu * n_cu;
}

hipError_t launch_join_small(hipStream_t stream, int n_cu, const int64_t* rpe_off,
                             const int32_t* rpe_ids, const uint16_t* rpe_cnt, int64_t n_blocks,
                             int32_t m, int32_t max_set, const int32_t* queries, int64_t n_queries,
                             int32_t k, int64_t* join_off, int64_t cap_rows, int32_t* out_ids,
                             uint16_t* out_cnt, uint16_t absent16, void* small_scan,
                             uint32_t spin_limit, int64_t* h_total, hipEvent_t done, uint32_t* err) {
    JoinJob j{};
    j.stream = stream, j.n_cu = n_cu;
    j.rpe_off = rpe_off, j.rpe_ids = rpe_ids, j.rpe_cnt = rpe_cnt, j.n_blocks = n_blocks, j.m = m;
    j.max_set = max_set, j.queries = queries, j.n_queries = n_queries, j.join_off_out = join_off;
    j.cap_rows = cap_rows, j.out_ids = out_ids, j.out_cnt = out_cnt, j.absent16 = absent16;
    j.small_scan = static_cast<SmallScan*>(small_scan), j.spin_limit = spin_limit;
    j.h_total = h_total, j.done = done, j.err = err;
    if (k == 2) return launch_join_lt<2, true>(j);
    if (k == 3) return launch_join_lt<3, true>(j);
    return hipErrorInvalidValue;
}

size_t small_scan_bytes() { return sizeof(SmallScan); }

}  // namespace surel
