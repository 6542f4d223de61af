// The fused walk + RPE kernel (walk_rpe_kernel.h): the forms without look-ups, and which form a call takes.
#include "walk_rpe_kernel.h"

namespace surel {

hipError_t launch_walk_rpe(hipStream_t stream, int max_lds_bytes, int n_cu, const int32_t* row_ptr,
                           const int32_t* col_idx, int32_t n_nodes, int64_t n_edges,
                           const int32_t* seeds, int64_t n_seeds, int32_t M, int32_t m,
                           uint64_t rng_seed, int32_t* walks, int64_t cap_rows, int64_t* rpe_off,
                           int32_t* ids, uint16_t* cnt, const EdgeRecords& rec, uint64_t* lb,
                           uint32_t spin_limit, int64_t* h_total, uint32_t* err, int32_t* code,
                           const PruneScratch& ps) {
    const FusedJob f = fused_job(row_ptr, col_idx, n_nodes, n_edges, seeds, n_seeds, M, m, rng_seed,
                                 walks, cap_rows, rpe_off, ids, cnt, rec, spin_limit, h_total, err);
    if (code == nullptr)
        return launch_walk_rpe_form<false>(stream, max_lds_bytes, n_cu, f, rec.format, lb, nullptr, VectorSet{});
    return launch_walk_rpe_codes(stream, max_lds_bytes, n_cu, f, rec.format, lb, code,
                                 vector_set(ps, spin_limit, err));
}

}  // namespace surel
