// The large-M kernel (gemm_big_kernel.h) with tiles of 192 rows.
#include "gemm_big_kernel.h"

namespace mlr {

template <int BITS, bool F16>
static hipError_t launch_192_dir(const GemmArgs &a, const BigPlan &plan, hipStream_t stream) {
    return a.backward ? launch_big_mt<BITS, true, F16, 192>(a, plan, stream) : launch_big_mt<BITS, false, F16, 192>(a, plan, stream);
}
template <bool F16>
static hipError_t launch_192_any(const GemmArgs &a, const BigPlan &plan, hipStream_t stream) {
    switch (a.w.bits) {
        case 2: return launch_192_dir<2, F16>(a, plan, stream);
        case 3: return launch_192_dir<3, F16>(a, plan, stream);
        default: return launch_192_dir<4, F16>(a, plan, stream);
    }
}
hipError_t launch_big_192(const GemmArgs &a, bool f16, const BigPlan &plan, hipStream_t stream) {
    return f16 ? launch_192_any<true>(a, plan, stream) : launch_192_any<false>(a, plan, stream);
}

}  // namespace mlr
