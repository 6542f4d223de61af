// The walker (Sec. 3.2 "Walk Sampling"; Algorithm 1, walk step): one lane moves one walk of
// m steps.  Shared by the stand-alone walk kernel and the fused walk + RPE kernel.
#pragma once

#include "device_util.h"

namespace surel {

// Per-edge neighbour records: one record per CSR entry e with the neighbour col_idx[e], the start
// of that neighbour's row and its degree, so that a step is one gather instead of two dependent
// ones.  Three layouts:
//   kRecPacked  one 64-bit word, id in the low id_bits, row start in the next lo_bits, degree in
//               the rest; id = n_nodes marks a bad entry, a degree field of all ones means "does
//               not fit, it is row_ptr[id + 1] - row start".  id_bits + lo_bits >= 32: the degree
//               lies in the upper half of the word;
//   kRecWide    int4 (id, row start, degree, 0); id -1 for an entry that names no node or whose
//               row is malformed: for graphs whose ids and row starts leave the packed degree too
//               few bits;
//   kRecShort   the id alone, id_bits <= 19 bits after id_bits bits, n_nodes marking a bad entry; the row
//               is looked up in row_ptr after all, except behind the last step.  For graphs of so few
//               nodes that row_ptr lies in every L2, and so many entries that packed records do not:
//               a line from memory carries 54 neighbours and more instead of 16, and a larger part of
//               the array stays in the L2 (see edge_record_plan).
constexpr int kRecNone = 0, kRecWide = 1, kRecPacked = 2, kRecShort = 3;

// Bits of the degree field of a packed record: what the two other fields leave, 31 at most.
__host__ __device__ constexpr int rec_degree_bits(int id_bits, int lo_bits) {
    return 64 - id_bits - lo_bits < 31 ? 64 - id_bits - lo_bits : 31;
}

// The graph as a walker sees it: the CSR, and optionally the records in one of the layouts.
struct WalkGraph {
    const int32_t* __restrict__ row_ptr;
    const int32_t* __restrict__ col_idx;
    const void* __restrict__ rec;
    int id_bits, lo_bits;  // kRecPacked; kRecShort: id_bits only
    int32_t n_nodes;
    int64_t n_edges;
};

// Both ends of node t's row in one load.
__device__ __forceinline__ void row_ends(const int32_t* __restrict__ row_ptr, uint32_t t, int32_t* lo,
                                         int32_t* hi) {
    typedef int ends_t __attribute__((ext_vector_type(2), aligned(4)));
    const ends_t ends = *reinterpret_cast<const ends_t*>(row_ptr + t);
    *lo = ends.x;
    *hi = ends.y;
}

// Row of the seed (wave-uniform loads); a malformed row counts as degree 0.
__device__ __forceinline__ bool seed_row(const WalkGraph& g, int32_t u, int32_t* lo, int32_t* deg) {
    const int32_t a = g.row_ptr[u];
    const int32_t d = g.row_ptr[u + 1] - a;
    const bool bad = a < 0 || d < 0 || (int64_t)a + d > g.n_edges;
    *lo = a;
    *deg = bad ? 0 : d;
    return bad;
}

// C walks of seed u per lane, moved in lock step so that a lane has C independent gathers in
// flight (the walk is bound by memory latency).  Walk c is number w[c], takes part if
// active[c], writes positions 0..m into row[c][0..m] (LDS rows of the lane's own) and calls
// visit(c, node) after every step.  Inactive walks still write a row (all u) that the caller
// ignores.  Step s uses word (s-1)&3 of Philox(counter (u, w, (s-1)>>2, 0), key).
// Returns true if a malformed CSR row or a neighbour id outside the graph was met (the
// walker then stays in place for that step).
// With records nothing here branches on the lane: a walker that does not move (no neighbours, or
// inactive, which is the same thing to it) reads record 0 and keeps its state by selects.
template <int kRec, int C, bool kPeel = true, typename Visit>
__device__ __forceinline__ bool walk_many(const WalkGraph& g, int32_t u, int32_t u_lo, int32_t u_deg,
                                          const int (&w)[C], const bool (&active)[C], int m,
                                          uint32_t key0, uint32_t key1, int32_t* const (&row)[C],
                                          Visit&& visit) {
    bool bad_graph = false;
    int32_t cur[C];
    uint32_t cur_lo[C], cur_deg[C];  // row of `cur`, of degree 0 if the walker does not move (kRec only)
#pragma unroll
    for (int c = 0; c < C; ++c) {
        cur[c] = u;
        cur_lo[c] = (uint32_t)u_lo;
        cur_deg[c] = active[c] ? (uint32_t)u_deg : 0u;
        row[c][0] = u;
    }
    // One group of four steps (one Philox call).  The first group is written out on its own:
    // there s0 is the constant 1, so the steps' row offsets and the Philox counter are known
    // at compile time (walks of up to four steps never leave it).  kPeel false: not written out,
    // which is half the code.
    auto group = [&](const int s0) __attribute__((always_inline)) {
        uint32_t r[C][4];
#pragma unroll
        for (int c = 0; c < C; ++c)
            philox4x32_10((uint32_t)u, (uint32_t)w[c], (uint32_t)((s0 - 1) >> 2), 0u, key0, key1,
                          r[c]);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int s = s0 + j;
            if (s <= m) {
                if (kRec != kRecNone) {
                    uint32_t e[C];
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        const uint32_t pick = mod_u32(r[c][j], max(cur_deg[c], 1u));
                        e[c] = cur_deg[c] != 0u ? cur_lo[c] + pick : 0u;
                    }
                    uint32_t id[C], lo[C], deg[C];
                    if (kRec == kRecWide) {
                        const int4* rec = static_cast<const int4*>(g.rec);
                        int4 nb[C];
#pragma unroll
                        for (int c = 0; c < C; ++c) nb[c] = rec[e[c]];
#pragma unroll
                        for (int c = 0; c < C; ++c) {
                            id[c] = (uint32_t)nb[c].x;  // -1: not below n_nodes
                            lo[c] = (uint32_t)nb[c].y;
                            deg[c] = (uint32_t)nb[c].z;
                        }
                    } else if (kRec == kRecShort) {
                        const char* rec = static_cast<const char*>(g.rec);
                        struct __attribute__((packed)) word_t { uint32_t v; };
#pragma unroll
                        for (int c = 0; c < C; ++c) {  // a record ends within four bytes of where it begins
                            const uint32_t bit = (uint32_t)__umul24(e[c], (uint32_t)g.id_bits);
                            const uint32_t word = reinterpret_cast<const word_t*>(rec + (bit >> 3))->v;
                            id[c] = __builtin_amdgcn_ubfe(word, bit & 7u, (uint32_t)g.id_bits);
                        }
#pragma unroll
                        for (int c = 0; c < C; ++c) lo[c] = deg[c] = 0u;
                        if (s < m) {  // nobody steps on from the last node
                            int32_t first[C], end[C];
#pragma unroll
                            for (int c = 0; c < C; ++c)
                                row_ends(g.row_ptr, min(id[c], (uint32_t)g.n_nodes - 1u), &first[c], &end[c]);
#pragma unroll
                            for (int c = 0; c < C; ++c) {
                                lo[c] = (uint32_t)first[c];
                                deg[c] = (uint32_t)(end[c] - first[c]);
                            }
                        }
                    } else {
                        const uint2* rec = static_cast<const uint2*>(g.rec);
                        const uint32_t id_mask = (1u << g.id_bits) - 1u;
                        const uint32_t lo_mask = (1u << g.lo_bits) - 1u;  // lo_bits <= 31
                        const uint32_t deg_shift = (uint32_t)(g.id_bits + g.lo_bits - 32);
                        const uint32_t deg_big = (1u << rec_degree_bits(g.id_bits, g.lo_bits)) - 1u;
                        uint2 nb[C];
#pragma unroll
                        for (int c = 0; c < C; ++c) nb[c] = rec[e[c]];
#pragma unroll
                        for (int c = 0; c < C; ++c) {
                            id[c] = nb[c].x & id_mask;
                            lo[c] = __builtin_amdgcn_alignbit(nb[c].y, nb[c].x, (uint32_t)g.id_bits) & lo_mask;
                            deg[c] = (nb[c].y >> deg_shift) & deg_big;
                            // a degree too large for its field: the record's row was validated
                            // when the records were made, so its end can be taken from the CSR
                            if (deg[c] == deg_big && id[c] < (uint32_t)g.n_nodes)
                                deg[c] = (uint32_t)g.row_ptr[id[c] + 1] - lo[c];
                        }
                    }
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        const bool go = cur_deg[c] != 0u;
                        const bool ok = id[c] < (uint32_t)g.n_nodes;
                        bad_graph = bad_graph || (go && !ok);
                        const bool move = go && ok;
                        cur[c] = move ? (int32_t)id[c] : cur[c];
                        cur_lo[c] = move ? lo[c] : cur_lo[c];
                        cur_deg[c] = move ? deg[c] : cur_deg[c];
                    }
                } else {
                    int32_t lo[C], hi[C];
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        lo[c] = 0;
                        hi[c] = 0;
                        if (active[c]) {
                            lo[c] = g.row_ptr[cur[c]];
                            hi[c] = g.row_ptr[cur[c] + 1];
                        }
                    }
                    int32_t nxt[C];
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        nxt[c] = cur[c];
                        if (lo[c] < 0 || hi[c] < lo[c] || (int64_t)hi[c] > g.n_edges) {
                            bad_graph = true;
                        } else if (hi[c] > lo[c]) {
                            const uint32_t deg = (uint32_t)(hi[c] - lo[c]);
                            nxt[c] = g.col_idx[(int64_t)lo[c] + (int64_t)mod_u32(r[c][j], deg)];
                        }
                    }
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        if ((uint32_t)nxt[c] >= (uint32_t)g.n_nodes) {
                            bad_graph = true;
                        } else {
                            cur[c] = nxt[c];
                        }
                    }
                }
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    row[c][s] = cur[c];
                    visit(c, cur[c]);
                }
            }
        }
    };
    if constexpr (kPeel) group(1);
    for (int s0 = kPeel ? 5 : 1; s0 <= m; s0 += 4) group(s0);
    return bad_graph;
}

}  // namespace surel
