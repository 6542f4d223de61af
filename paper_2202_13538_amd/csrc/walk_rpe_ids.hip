// The fused walk + RPE kernel (walk_rpe_kernel.h): the forms that look every row's vector up as well.
#include "walk_rpe_kernel.h"

namespace surel {

hipError_t launch_walk_rpe_codes(hipStream_t stream, int max_lds_bytes, int n_cu, const FusedJob& f,
                                 int rec_format, uint64_t* lb, int32_t* code, const VectorSet& set) {
    return launch_walk_rpe_form<true>(stream, max_lds_bytes, n_cu, f, rec_format, lb, code, set);
}

}  // namespace surel
