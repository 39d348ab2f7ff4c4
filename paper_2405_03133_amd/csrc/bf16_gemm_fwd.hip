// Forward GEMM instantiations: gate/up projections with the SwiGLU epilogue,
// and the down projection.
#include "bf16_kernels.h"

namespace lory {
namespace k {

hipError_t launch_gu(hipStream_t st, const gemm::Params &p, const EpiGU &d)
{
    // A = X_s [T][d] (K contiguous), B = merged slabs [d][nf] (N contiguous), two sets.
    // Two output modes: G and U (the activation is then a streaming pass over them), or the
    // activation alone.  A three-plane epilogue (G, U and A at once) is not instantiated: it needs
    // scratch memory for spilled registers and measured slower than the separate pass.
    const bool save = d.G != nullptr, act = d.Act != nullptr;
    if (save == act) return hipErrorInvalidValue;
    if (act) {
        const EpiGUT<false, true> e = {d.G, d.U, d.Act, d.T, d.dff, d.n_off};
        return gemm2::launch_rows<2, 1, false, true>(p, e, st);
    }
    const EpiGUT<true, false> e = {d.G, d.U, d.Act, d.T, d.dff, d.n_off};
    return gemm2::launch_rows<2, 1, false, true>(p, e, st);
}

hipError_t launch_gu2(hipStream_t st, const gemm::Params &p, const EpiAct2 &e)
{
    return gemm2::launch_rows<2, 1, false, true>(p, e, st);
}

hipError_t launch_down(hipStream_t st, const gemm::Params &p, const EpiStore &e)
{
    // A = Act_s [T][d_ff], B = merged slab [d_ff][jf] (N contiguous)
    return gemm2::launch_rows<1, 1, false, true>(p, e, st);
}

hipError_t launch_down2(hipStream_t st, const gemm::Params &p, const EpiStore &e)
{
    // A = the two terms of Act_s, both with the same merged slab
    return gemm2::launch_rows<1, 2, false, true>(p, e, st);
}

hipError_t launch_gu_split(hipStream_t st, const gemm::Params &p, const EpiPart<2> &e, int rows)
{
    if (rows == 128) return gemm2::launch<2, 1, false, true, gemm2::T128>(p, e, st);
    return gemm2::launch<2, 1, false, true, gemm2::T64>(p, e, st);
}

hipError_t launch_down_split(hipStream_t st, const gemm::Params &p, const EpiPart<1> &e, int rows)
{
    if (rows == 128) return gemm2::launch<1, 1, false, true, gemm2::T128>(p, e, st);
    return gemm2::launch<1, 1, false, true, gemm2::T64>(p, e, st);
}

}  // namespace k
}  // namespace lory
