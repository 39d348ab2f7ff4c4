// Backward weight GEMM instantiations (contraction over the T tokens of a
// segment): dWg_bar = X^T dG and dWu_bar = X^T dU share X; dWd_bar = A^T dY.
#include "bf16_kernels.h"

namespace lory {
namespace k {

hipError_t launch_dwgu(hipStream_t st, const gemm::Params &p, const EpiStore2 &e)
{
    // A = X_s stored [T][d] (M contiguous), B = dG_s / dU_s stored [T][d_ff] (N contiguous).
    // The contraction is only T long, so the kernel is bound by writing its output: sharing X
    // between the two operand sets saves little, and two single-set launches (256-wide rows of
    // output per wave pair, half as many stores in flight per tile) measured a little faster - unless the tiles of
    // both fit one round of the CUs, where a launch is what a call costs (8 segments of 64 tokens at d = d_ff = 64: 9.6
    // us in two launches, 5.1 in one).
    if (gemm2::rounds_of(p, 128, 128) <= 1.0) return gemm2::launch<2, 1, true, true, gemm2::W128>(p, e, st);
    gemm::Params q = p;
    EpiStore e0 = {e.C0, e.c_batch, e.ldc};
    hipError_t rc = launch_dwd(st, q, e0);
    if (rc != hipSuccess) return rc;
    q.B[0] = p.B[1]; q.b_batch[0] = p.b_batch[1]; q.ldb[0] = p.ldb[1];
    EpiStore e1 = {e.C1, e.c_batch, e.ldc};
    return launch_dwd(st, q, e1);
}

hipError_t launch_dwd(hipStream_t st, const gemm::Params &p, const EpiStore &e)
{
    // A = Act_s stored [T][d_ff] (M contiguous), B = dY_s stored [T][d] (N contiguous)
    return gemm2::launch_weight<1, 1, true, true>(p, e, st);
}

}  // namespace k
}  // namespace lory
