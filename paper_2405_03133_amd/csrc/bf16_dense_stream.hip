// Dense FFN of few token rows per sequence: plans and launches of the streaming projections.
#include "dense_stream_bf16.h"

namespace lory {
namespace k {

namespace {

constexpr int kGuWaves = 4, kDownWaves = 8;
constexpr size_t kMaxActLds = 96 * 1024;

// K slices of a projection whose unsplit form has `wgs` workgroups of `steps` K steps: the estimate is rounds of
// workgroups over the CUs times the time of one, `u` us for a K step of each of its wavefronts and 2.4 for its start
// and its sums.  More workgroups than CUs pay for the last, partly empty round although several share a CU: 4 sequences
// at d = 2112, d_ff = 5056, gate/up in 320 / 640 / 960 workgroups 58.3 / 54.6 / 53.5 us; 2 at 1216, 4992 in
// 156 / 312 / 468 20.1 / 21.6 / 20.0.  per_slice: us that the partial sums of a slice cost their reader; once: of the
// launch that adds them.
int slices(long wgs, int steps, int waves, double u, double per_slice, double once, int min_ks, size_t max_ks)
{
    const int cus = gemm2::cu_count();
    int best = 0;
    double best_t = 0;
    for (int ks = min_ks; ks <= steps && (size_t)ks <= max_ks && (ks == min_ks || wgs * ks <= 4L * cus); ++ks) {
        const int s = (steps + ks - 1) / ks;
        const double rounds = (double)((wgs * ks + cus - 1) / cus);
        const double wave_steps = 0.5 * ((s + waves - 1) / waves + (double)steps / ks / waves);
        const double t = rounds * (wave_steps * u + 2.4) + ks * per_slice + (ks > 1 ? once : 0.0);
        if (!best || t < best_t) {
            best = ks;
            best_t = t;
        }
    }
    return best;
}

}  // namespace

DenseStream dense_stream_plan(int B, int M, int d, int dff, size_t floats)
{
    DenseStream p = {0, 0};
    if (M > stream::kMaxRows || B > 32767 || d >= (1 << 26) || dff >= (1 << 26)) return p;
    const long cg = (dff + stream::kCols - 1) / stream::kCols, cd = (d + stream::kCols - 1) / stream::kCols;
    const size_t fg = (size_t)2 * B * M * dff, fd = (size_t)B * M * d;
    if (floats < fg + fd) return p;
    // the activation of a slice has to fit in LDS
    const int dsteps = dff / 32;
    int min_d = 1;
    while (stream::lds_bytes<true, kDownWaves>(M, dsteps, min_d) > kMaxActLds) ++min_d;
    // every column block of the down projection reads the gate/up sums of its rows again, from L2
    p.gu = slices(2 * B * cg, d / 32, kGuWaves, 1.2, 4.0 * fg * cd / 8e6, 0.0, 1, (floats - fd) / fg);
    p.down = slices(B * cd, dsteps, kDownWaves, 2.2, 8.0 * fd / 5e6, 4.5, min_d, (floats - p.gu * fg) / fd);
    if (!p.down) p.gu = 0;
    return p;
}

int dense_stream_gu_slices(int B, int M, int d, int dff, size_t floats)
{
    if (M <= stream::kMaxRows || M > stream::kMaxGuRows || B > 32767 || d >= (1 << 26) || dff >= (1 << 26)) return 0;
    const long cols = (dff + stream::kCols - 1) / stream::kCols;
    const size_t fg = (size_t)2 * B * M * dff;
    if (floats < fg) return 0;
    // every sum is written once and read once
    return slices(2 * B * cols, d / 32, kGuWaves, 1.2, 8.0 * fg / 12e6, 0.0, 1, floats / fg);
}

hipError_t launch_dense_stream_gu(hipStream_t st, const stream::Params &p, int B)
{
    if (p.M <= 16) return stream::launch<false, kGuWaves, 2>(st, p, B);
    if (p.M <= 32) return stream::launch<false, kGuWaves, 2, 2>(st, p, B);
    if (p.M <= 48) return stream::launch<false, kGuWaves, 2, 3>(st, p, B);
    return stream::launch<false, kGuWaves, 2, 4>(st, p, B);
}

hipError_t launch_dense_stream_down(hipStream_t st, const stream::Params &p, int B)
{
    return stream::launch<true, kDownWaves, 2>(st, p, B);
}

}  // namespace k
}  // namespace lory
