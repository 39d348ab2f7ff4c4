// Backward data GEMM instantiations: dA = dY Wd_bar^T and dX = dG Wg_bar^T + dU Wu_bar^T.
#include "bf16_kernels.h"

namespace lory {
namespace k {

hipError_t launch_da(hipStream_t st, const gemm::Params &p, const EpiStore &e)
{
    // A = dY_s [T][d], B = merged slab rows [nf][d] (K contiguous)
    return gemm2::launch_rows<1, 1, false, false>(p, e, st);
}

hipError_t launch_dx(hipStream_t st, const gemm::Params &p, const EpiStore &e)
{
    // two sources: (dG_s, Wg_bar rows [kf][d_ff]) and (dU_s, Wu_bar rows), all K contiguous
    return gemm2::launch_rows<1, 2, false, false>(p, e, st);
}

}  // namespace k
}  // namespace lory
