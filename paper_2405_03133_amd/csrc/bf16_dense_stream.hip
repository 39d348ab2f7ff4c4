// Dense FFN of few token rows per sequence: plans and launches of the streaming projections.
#include "dense_stream_bf16.h"

#include <math.h>

namespace lory {
namespace k {

namespace {

constexpr int kGuWaves = 4, kDownWaves = 8;
constexpr size_t kMaxActLds = 96 * 1024;

// K slices that are tried; more workgroups than four for each CU are not.
constexpr int kLadder[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32};

bool fits(long wgs, int ks) { return ks == 1 || wgs * ks <= 4L * gemm2::cu_count(); }

// More workgroups than CUs pay for the last, partly empty round although several share a CU: 4 sequences
// at d = 2112, d_ff = 5056, gate/up in 320 / 640 / 960 workgroups 58.3 / 54.6 / 53.5 us; 2 at 1216, 4992 in
// 156 / 312 / 468 20.1 / 21.6 / 20.0.
double rounds(long wgs) { return (double)((wgs + gemm2::cu_count() - 1) / gemm2::cu_count()); }

// K steps of a wavefront: between the most that one has and their mean
double wave_steps(int steps, int ks, int waves)
{
    return 0.5 * (((steps + ks - 1) / ks + waves - 1) / waves + (double)steps / ks / waves);
}

}  // namespace

// Up to 16 rows.  The slices of both projections are chosen together, because each column block of the down projection
// reads the gate/up sums of its rows, slice by slice, four at a time and 512 quads of the activation at a time, before it
// starts.  Estimated us of a form: rounds of workgroups over the CUs times a wavefront's K steps and the start of one
// (down: with the activation), the sums of gate/up written and read again, and for a cut down projection the launch
// that adds.  Fitted to 41 forms each of 378 calls (1 .. 12 sequences of 1 .. 16 rows, d = 768 .. 2560): 0.9 % slower than
// the fastest form of a call on average, 10 % at most (the slices chosen one after the other, without the rounds of
// reading: 2.2 and 43; 16 rows at d = 2048, d_ff = 704 18.9 us, now 13.2).
DenseStream dense_stream_plan(int B, int M, int d, int dff, size_t floats)
{
    DenseStream best = {0, 0};
    if (M > stream::kMaxRows || B > 32767 || d >= (1 << 26) || dff >= (1 << 26)) return best;
    const long cg = (dff + stream::kCols - 1) / stream::kCols, cd = (d + stream::kCols - 1) / stream::kCols;
    const size_t fg = (size_t)2 * B * M * dff, fd = (size_t)B * M * d;
    // the activation of a slice has to fit in LDS
    const int gsteps = d / 32, dsteps = dff / 32;
    int min_d = 1;
    while (stream::lds_bytes<true, kDownWaves>(M, dsteps, min_d) > kMaxActLds) ++min_d;
    double best_t = 0;
    for (int g : kLadder) {
        if (g > gsteps || g * fg + fd > floats || !fits(2 * B * cg, g)) break;
        const double tg = rounds(2 * B * cg * g) * (wave_steps(gsteps, g, kGuWaves) * 0.88 + 0.65) + (double)(g * fg) * (0.5e-6 + 0.6e-6 * cd);
        for (int k : kLadder) {
            if (k < min_d) k = min_d;
            if (k > dsteps || (k > min_d && !fits(B * cd, k)) || (size_t)k > (floats - g * fg) / fd) break;
            const double quads = M * 8.0 * ((dsteps + k - 1) / k);
            const double act = ceil(quads / 512) * (0.64 * ((g + 3) / 4) + 0.4);
            const double t = tg + rounds(B * cd * k) * (wave_steps(dsteps, k, kDownWaves) * 0.89 + 1.2 + act) +
                             (k > 1 ? 1.3 + 6e-6 * k * fd : 0.0);
            if (!best.gu || t < best_t) {
                best = {g, k};
                best_t = t;
            }
        }
    }
    return best;
}

// Gate/up alone: its K slices, or 0 where the ring GEMM, which is estimated to take ring_us for the contraction, is not
// slower.  The estimate: rounds of workgroups over the CUs times a wavefront's K steps and the sums of the rows, and more
// the more CUs share the memory in the last round.  Fitted, with the ring GEMM's, to the differences of 346 calls (1 .. 12
// sequences of 17 .. 63 rows, d = 768 .. 2560) that the ring GEMM would cut: a call takes 0.949 of the ring GEMM's time on
// average and 0.5 % more than the better of the two, 9 % at most (2 x 49 rows at d = 1024, d_ff = 2816 34.3 us, ring 31.5);
// streamed in all of them, in slices chosen for the read rate alone, 0.958, 1.4 % and 13 % (12 x 63 at 2048, 704 50.2 us, ring 44.6).
int dense_stream_gu_slices(int B, int M, int d, int dff, size_t floats, double ring_us)
{
    if (M <= stream::kMaxRows || M > stream::kMaxGuRows || B > 32767 || d >= (1 << 26) || dff >= (1 << 26)) return 0;
    const long wgs = 2L * B * ((dff + stream::kCols - 1) / stream::kCols), cus = gemm2::cu_count();
    const size_t fg = (size_t)2 * B * M * dff;
    int best = 0;
    double best_t = 0.955 * ring_us;
    for (int ks : kLadder) {
        if (ks > d / 32 || ks * fg > floats || !fits(wgs, ks)) break;
        const double last = (double)((wgs * ks - 1) % cus + 1) / cus;
        const double t = rounds(wgs * ks) * (wave_steps(d / 32, ks, kGuWaves) * 0.92 + 3.3 + 0.04 * M) + 5.5 * last;
        if (t < best_t) {
            best = ks;
            best_t = t;
        }
    }
    return best;
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
