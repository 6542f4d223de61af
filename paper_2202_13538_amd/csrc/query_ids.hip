// Query-level RPE-IDs per walk position (Sec. 3.4, the form the section describes first): the
// walks W_u, u in Q, are concatenated and every node occurrence x in them gets
// RPE-ID_{Q,x} = [RPE-ID_{u,x}]_{u in Q}.  The RPE table is the (unpruned) central array of
// Sec. 3.3, so RPE-ID_{u,x} is the index of (u, x)'s row in it; -1 stands for "x is not in
// V_u" (the all-zero vector).  The paper looks x up in the hash dictionary H_u.
//
// Here the blocks' id lists are sorted, and a workgroup (one to four wavefronts, by the length of
// the walk blocks) stages the K lists of a query in LDS with a directory for each: the range of
// the list's ids cut into as many equal parts as the list may have ids (a power of two), and for
// every part the place of the first id in it or behind it.  A look-up reads the directory and
// then the list from there on: one or two ids, since node ids lie evenly in their range wherever
// labels carry no order.  The 2K directory entries and first ids of an entry's look-ups are read
// for all entries of a thread together; only lanes that have to go on read further.  Lists whose
// ids crowd together (more than kCrowd in one part) are searched by bisection instead, which needs
// no directory.
// What bounds it: LDS reads at random places (a wavefront's 64 lanes hit some banks four or five
// times) and the instructions around them, so that waves in flight are what counts: 65,536 pairs of
// M = 200, m = 4 with codes take 0.43 ms (5.0 TB/s of the bytes in and out; 0.46 when the results
// went through the caches) with eight waves per SIMD, 0.50 with five; twice as many parts, 0.55; a
// wave per query with bisection, 1.22.
// (Per-query hash dictionaries in LDS were measured too and lost: their probe loops diverge.)
#include "device_util.h"
#include "kernels.h"

namespace surel {

// The K row indices of one walk entry (4-byte aligned, written with one store).
template <int K>
struct RowIds {
    typedef int32_t type __attribute__((ext_vector_type(K), aligned(4)));
};

constexpr int kCrowd = 8;  // ids in one part of the directory, at most
constexpr uint32_t kQidEnd = 0xFFFFFFFFu;

// LDS of one workgroup, in 32-bit words.
struct QidLds {
    int list;     // words from one list's ids to the next one's
    int codes;    // first list's codes
    int dir;      // first list's directory (16-bit entries)
    int parts;    // entries of a directory, a power of two
    int total;
};
__host__ __device__ inline QidLds qid_lds(int K, int max_set, bool code) {
    QidLds o;
    o.list = max_set + 2;  // behind the last id: two that no walk entry reaches
    o.codes = K * o.list;
    o.dir = o.codes * (code ? 2 : 1);
    o.parts = 64;
    while (o.parts < max_set && o.parts < 2048) o.parts *= 2;
    o.total = o.dir + K * o.parts / 2;
    return o;
}

template <int K>
__device__ __forceinline__ int n_of(const int (&n)[K], int j) {
    int v = n[0];
#pragma unroll
    for (int jj = 1; jj < K; ++jj) v = j == jj ? n[jj] : v;
    return v;
}

// kQiEntries: walk entries of a block that a thread looks up at a time.
// kCode: the rows' codes (their RPE-IDs in the pruned array of Sec. 3.3) are staged next to the
// ids and go out instead of the row indices.
template <int K, int kQiEntries, bool kCode>
__global__ __launch_bounds__(256, 8) void query_ids_kernel(
    const int32_t* __restrict__ walks, const int64_t* __restrict__ rpe_off,
    const int32_t* __restrict__ rpe_ids, const int32_t* __restrict__ code, int64_t n_blocks,
    int32_t n_key, int32_t max_set, int64_t table_rows, const int32_t* __restrict__ queries,
    int64_t n_queries, int32_t* __restrict__ out, uint32_t* __restrict__ err) {
    extern __shared__ __align__(16) uint32_t lds32[];
    __shared__ uint32_t crowded;
    const int T = (int)blockDim.x;
    const int tid = (int)threadIdx.x;
    const QidLds lay = qid_lds(K, max_set, kCode);
    uint16_t* const dirs = reinterpret_cast<uint16_t*>(lds32 + lay.dir);
    for (int64_t q = blockIdx.x; q < n_queries; q += gridDim.x) {
        // the K blocks of this query (the same in every thread)
        int32_t blk[K];
        int64_t lo[K];
        int n[K];
        uint32_t problem = 0;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int32_t b = queries[q * K + j];
            blk[j] = 0;
            lo[j] = 0;
            n[j] = 0;
            if (b < 0 || (int64_t)b >= n_blocks) {
                problem |= kDevBadQuery;
            } else {
                const int64_t a = rpe_off[b];
                const int64_t len = rpe_off[b + 1] - a;
                if (a < 0 || len < 0 || a + len > table_rows) {
                    problem |= kDevBadTable;
                } else if (len > (int64_t)max_set) {
                    problem |= kDevSetTooLarge;
                } else {
                    blk[j] = b;
                    lo[j] = a;
                    n[j] = (int)len;
                }
            }
        }
        int32_t* out_q = out + q * (int64_t)K * n_key * K;
        if (problem != 0) {
            // the query gets no RPE-IDs at all
            if (tid == 0) atomicOr(err, problem);
            for (int t = tid; t < K * n_key * K; t += T) out_q[t] = -1;
            continue;
        }
        // the first entries of every walk block (all of them, for the usual sizes) are asked for
        // before the id lists, so that one wait covers both
        uint32_t x_first[K][kQiEntries];
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int32_t* W = walks + (int64_t)blk[j] * n_key;
#pragma unroll
            for (int e = 0; e < kQiEntries; ++e)
                x_first[j][e] = (uint32_t)__builtin_nontemporal_load(W + min(e * T + tid, n_key - 1));
        }
        __syncthreads();  // the LDS words of the query before are free
        if (tid == 0) crowded = 0u;
        // every list's words, ids and codes, are asked for together
        constexpr int kStageU = 4;
        constexpr int kLists = kCode ? 2 * K : K;
        for (int t0 = 0; t0 < max_set; t0 += kStageU * T) {
            bool any = false;
#pragma unroll
            for (int j = 0; j < K; ++j) any = any || t0 < n[j];
            if (!any) break;
            uint32_t staged[kLists][kStageU];
#pragma unroll
            for (int l = 0; l < kLists; ++l) {
                const int32_t* from = (l < K ? rpe_ids : code) + lo[l % K];
#pragma unroll
                for (int u = 0; u < kStageU; ++u) {
                    const int t = t0 + u * T + tid;
                    staged[l][u] = t < n[l % K] ? (uint32_t)from[t] : 0u;
                }
            }
#pragma unroll
            for (int l = 0; l < kLists; ++l) {
                uint32_t* to = lds32 + (l < K ? 0 : lay.codes) + (l % K) * lay.list;
#pragma unroll
                for (int u = 0; u < kStageU; ++u) {
                    const int t = t0 + u * T + tid;
                    if (t < n[l % K]) to[t] = staged[l][u];
                }
            }
        }
        if (tid < 2 * K) lds32[(tid >> 1) * lay.list + n_of<K>(n, tid >> 1) + (tid & 1)] = kQidEnd;
        __syncthreads();
        // The directories.  x lies in part mulhi(x - first, scale) of its list's range; part p's
        // entry is the place of the first id in part p or behind it, so the thread of id t writes
        // the entries of the parts behind the one of id t - 1, up to its own.
        uint32_t first[K], range[K], scale[K];
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const uint32_t* ids = lds32 + j * lay.list;
            first[j] = n[j] > 0 ? ids[0] : 0u;
            range[j] = n[j] > 0 ? ids[n[j] - 1] - first[j] : 0u;
            // a little below parts * 2^32 / (range + 1), so that the last id's part is below
            // `parts`, in single precision (2^-20 covers its errors); ranges below `parts` share
            // the largest scale that fits 32 bits
            const float r1 = (float)max(range[j], (uint32_t)lay.parts) + 1.0f;
            scale[j] = (uint32_t)((float)lay.parts * 4294967296.0f * __builtin_amdgcn_rcpf(r1) *
                                  (1.0f - 0x1p-20f));
            uint16_t* dir = dirs + j * lay.parts;
            bool crowd = false;
            for (int t = tid; t < n[j]; t += T) {
                const uint32_t part = __umulhi(ids[t] - first[j], scale[j]);
                const int before = t > 0 ? (int)__umulhi(ids[t - 1] - first[j], scale[j]) : -1;
                crowd = crowd || (t >= kCrowd && __umulhi(ids[t - kCrowd] - first[j], scale[j]) == part);
                for (int p = max(before, -1) + 1; p <= (int)min(part, (uint32_t)lay.parts - 1u); ++p)
                    dir[p] = (uint16_t)t;
            }
            if (__ballot(crowd) != 0ull && (tid & (kWave - 1)) == 0) atomicOr(&crowded, 1u << j);
        }
        __syncthreads();
        const uint32_t bisect = crowded;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int32_t* W = walks + (int64_t)blk[j] * n_key;
            int32_t* out_j = out_q + (int64_t)j * n_key * K;
            for (int t0 = 0; t0 < n_key; t0 += kQiEntries * T) {
                uint32_t x[kQiEntries];
                uint32_t pos[kQiEntries][K];  // place in list j2 where the search ended
                uint32_t at[kQiEntries][K];   // the id there (kQidEnd behind the list)
#pragma unroll
                for (int e = 0; e < kQiEntries; ++e) {
                    const int t = min(t0 + e * T + tid, n_key - 1);
                    x[e] = t0 == 0 ? x_first[j][e] : (uint32_t)__builtin_nontemporal_load(W + t);
                    x[e] = min(x[e], kQidEnd - 1u);  // an entry of -1 names no node
                }
#pragma unroll
                for (int j2 = 0; j2 < K; ++j2) {
                    const uint32_t* ids = lds32 + j2 * lay.list;
                    const uint16_t* dir = dirs + j2 * lay.parts;
                    if ((bisect >> j2 & 1u) == 0u) {
                        // an id outside the list's range is looked up in the last part
                        bool more = false;
#pragma unroll
                        for (int e = 0; e < kQiEntries; ++e)
                            pos[e][j2] = dir[__umulhi(min(x[e] - first[j2], range[j2]), scale[j2])];
#pragma unroll
                        for (int e = 0; e < kQiEntries; ++e) {
                            pos[e][j2] = min(pos[e][j2], (uint32_t)n[j2]);
                            const uint32_t a0 = ids[pos[e][j2]], a1 = ids[pos[e][j2] + 1];
                            pos[e][j2] += a0 < x[e] ? 1u : 0u;
                            at[e][j2] = a0 < x[e] ? a1 : a0;
                            more = more || at[e][j2] < x[e];
                        }
                        while (more) {  // ends at kQidEnd
                            more = false;
#pragma unroll
                            for (int e = 0; e < kQiEntries; ++e) {
                                if (at[e][j2] < x[e]) at[e][j2] = ids[++pos[e][j2]];
                                more = more || at[e][j2] < x[e];
                            }
                        }
                    } else {
                        // pos = number of ids below x
                        for (int e = 0; e < kQiEntries; ++e) pos[e][j2] = 0u;
                        for (uint32_t step = 1u << (31 - __builtin_clz((unsigned)n[j2])); step > 0; step >>= 1) {
#pragma unroll
                            for (int e = 0; e < kQiEntries; ++e) {
                                const uint32_t cand = pos[e][j2] + step;
                                if (cand <= (uint32_t)n[j2] && ids[min(cand, (uint32_t)n[j2]) - 1u] < x[e])
                                    pos[e][j2] = cand;
                            }
                        }
#pragma unroll
                        for (int e = 0; e < kQiEntries; ++e) at[e][j2] = ids[pos[e][j2]];
                    }
                }
#pragma unroll
                for (int e = 0; e < kQiEntries; ++e) {
                    const int t = t0 + e * T + tid;
                    typename RowIds<K>::type row;
#pragma unroll
                    for (int j2 = 0; j2 < K; ++j2) {
                        const bool found = at[e][j2] == x[e];
                        if constexpr (kCode) {
                            row[j2] = -1;
                            if (found) row[j2] = (int32_t)lds32[lay.codes + j2 * lay.list + pos[e][j2]];
                        } else {
                            row[j2] = found ? (int32_t)((uint32_t)lo[j2] + pos[e][j2]) : -1;
                        }
                    }
                    // The K indices of an entry as one 4*K-byte store, past the caches for results of any
                    // size.  Through / past them, us: 64 pairs of M = 200, m = 4 (1 MB) 9.3 / 9.3, 2,048
                    // (33 MB) 20.4 / 17.3, 8,192 (131 MB) 58.9 / 58.8, 16,384 112 / 108, 65,536 412 / 398;
                    // triples of M = 61, m = 3, 8,192 of them (72 MB) 46.8 / 47.4, 65,536 289 / 273; 1,024
                    // pairs of M = 25, m = 2 6.2 / 6.5.  Whoever reads the results next takes as long, but
                    // for the 72 MB in buffers used in turn: 69.9 / 74.2 with a pass over them behind it.
                    if (t < n_key)
                        __builtin_nontemporal_store(
                            row, reinterpret_cast<typename RowIds<K>::type*>(out_j + (int64_t)t * K));
                }
            }
        }
    }
}

template <int K, int QE, bool kCode>
static hipError_t launch_query_ids_ke(hipStream_t stream, int threads, const int32_t* walks,
                                      const int64_t* rpe_off, const int32_t* rpe_ids,
                                      const int32_t* code, int64_t n_blocks, int32_t n_key,
                                      int32_t max_set, int64_t table_rows, const int32_t* queries,
                                      int64_t n_queries, int32_t* out, uint32_t* err) {
    const size_t lds_bytes = (size_t)qid_lds(K, max_set, kCode).total * 4;
    const void* fn = reinterpret_cast<const void*>(query_ids_kernel<K, QE, kCode>);
    if (lds_bytes > 48 * 1024) {
        hipError_t rc = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                            (int)lds_bytes);
        if (rc != hipSuccess) return rc;
    }
    // a workgroup per query and the hardware hands them out (a workgroup loops only where the grid
    // cannot be that large)
    const int64_t most = 0x7FFFFFFFll / threads;
    hipLaunchKernelGGL((query_ids_kernel<K, QE, kCode>),
                       dim3((unsigned)(n_queries < most ? n_queries : most)), dim3(threads), lds_bytes,
                       stream, walks, rpe_off, rpe_ids, code, n_blocks, n_key, max_set, table_rows,
                       queries, n_queries, out, err);
    return hipGetLastError();
}

// Up to four entries of a walk block a thread at a time, and as many wavefronts as then cover the
// block, four at most.
template <int K, bool kCode>
static hipError_t launch_query_ids_k(hipStream_t stream, const int32_t* walks, const int64_t* rpe_off,
                                     const int32_t* rpe_ids, const int32_t* code, int64_t n_blocks,
                                     int32_t n_key, int32_t max_set, int64_t table_rows,
                                     const int32_t* queries, int64_t n_queries, int32_t* out,
                                     uint32_t* err) {
#define SUREL_QI_LAUNCH(QE_, THREADS_)                                                          \
    return launch_query_ids_ke<K, QE_, kCode>(stream, THREADS_, walks, rpe_off, rpe_ids, code, \
                                              n_blocks, n_key, max_set, table_rows, queries,   \
                                              n_queries, out, err)
    if (n_key <= kWave) SUREL_QI_LAUNCH(1, 64);
    if (n_key <= 2 * kWave) SUREL_QI_LAUNCH(2, 64);
    if (n_key <= 4 * kWave) SUREL_QI_LAUNCH(4, 64);
    if (n_key <= 8 * kWave) SUREL_QI_LAUNCH(4, 128);
    SUREL_QI_LAUNCH(4, 256);
#undef SUREL_QI_LAUNCH
}

hipError_t launch_query_ids(hipStream_t stream, int max_lds_bytes, const int32_t* walks,
                            const int64_t* rpe_off, const int32_t* rpe_ids, const int32_t* code,
                            int64_t n_blocks, int32_t M, int32_t m, int32_t max_set,
                            int64_t table_rows, const int32_t* queries, int64_t n_queries, int32_t k,
                            int32_t* out, uint32_t* err) {
    if (n_queries == 0) return hipSuccess;
    if ((size_t)qid_lds(k, max_set, code != nullptr).total * 4 + 64 > (size_t)max_lds_bytes)
        return hipErrorInvalidValue;
    const int32_t n_key = M * (m + 1);
#define SUREL_QI_ARGS \
    stream, walks, rpe_off, rpe_ids, code, n_blocks, n_key, max_set, table_rows, queries, n_queries, out, err
    if (k == 2 && !code) return launch_query_ids_k<2, false>(SUREL_QI_ARGS);
    if (k == 3 && !code) return launch_query_ids_k<3, false>(SUREL_QI_ARGS);
    if (k == 2) return launch_query_ids_k<2, true>(SUREL_QI_ARGS);
    if (k == 3) return launch_query_ids_k<3, true>(SUREL_QI_ARGS);
#undef SUREL_QI_ARGS
    return hipErrorInvalidValue;
}

}  // namespace surel
