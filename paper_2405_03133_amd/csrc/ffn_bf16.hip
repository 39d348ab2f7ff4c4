// bf16 merged FFN forward and backward (paper Eq. 1 / Eq. 2, SwiGLU experts):
// host-side orchestration of the MFMA kernels.
//
// Unless the caller asks for them (Wbar_save: the forward then merges straight
// into the caller's buffer and the backward reads them there instead of
// re-merging), the merged parameters of all segments (S * 3 * d * d_ff values)
// are never held at once.  Each pass walks the expert matrices block by block; for a
// block it (1) merges that block for ALL segments into a bounded slab (one read
// of the expert stack, thin MFMA GEMM over the E experts), (2) runs the
// per-segment token GEMMs that consume the slab.  The backward additionally
// produces per-segment weight-gradient slabs that the scatter kernel folds
// into the E expert gradients and into the router-weight gradients at once.
// The slab budget (default 6 GiB) trades workspace for launch size: blocks large enough to
// fill all 256 CUs several times over measured faster than cache-sized blocks.
#include "lory_internal.h"

#include <stdlib.h>

#include "bf16_kernels.h"

namespace lory {

namespace {

using gemm::Params;
using k::EpiGU;
using k::EpiStore;
using k::EpiStore2;
using ms::MergeParams;
using ms::Rect;
using ms::ScatterParams;

typedef uint16_t bf;

size_t g_slab_budget = 0;  // 0 = not initialised yet

size_t slab_budget_bytes()
{
    if (g_slab_budget == 0) {
        size_t mb = 6144;
        if (const char *env = getenv("LORY_SLAB_MB")) {
            const long v = atol(env);
            if (v >= 1 && v <= 16384) mb = (size_t)v;
        }
        g_slab_budget = mb << 20;
    }
    return g_slab_budget;
}

// Which token contractions run with the merge inside the GEMM (fused_bf16.h) instead of the slab pipeline: 0 none, 1 those
// that are estimated to be faster (fused_pays), 2 all wherever the shape fits the kernel, 3 like 2 and with the
// backward's per-segment weight gradients kept on chip as well (fsg_kernel; measured slower than the
// slab pipeline at every shape tried, so no other mode uses it).
int g_fused_mode = -1;  // -1 = not initialised yet

int fused_mode()
{
    if (g_fused_mode < 0) {
        int mode = 1;
        if (const char *env = getenv("LORY_FUSED")) {
            const long v = atol(env);
            if (v >= 0 && v <= 3) mode = (int)v;
        }
        g_fused_mode = mode;
    }
    return g_fused_mode;
}

fmg::Params fused_params(const Dims &m, const bf *A0, const bf *A1, int lda, const bf *W0, const bf *W1, int ldw,
                         const float *w, int N, int K, bf *C, int ldc)
{
    fmg::Params p = {};
    p.A[0] = A0; p.A[1] = A1; p.lda[0] = p.lda[1] = lda;
    p.W[0] = W0; p.W[1] = W1;
    p.expert_stride = m.D; p.ldw = ldw;
    p.w = w; p.E = m.E; p.T = m.T; p.tokens = (int)m.tokens;
    p.N = N; p.K = K; p.C = C; p.ldc = ldc;
    return p;
}

// The contractions of the layer that are merged inside the GEMM.
struct Fused {
    bool gate_up, down, da, dx;
};

// Whether the merge inside the GEMM is estimated to be faster for a contraction of `mats` expert matrices (two operand sets
// or two sources) with N output columns and K per source: on the eight-wave kernel (segments of 64 or 128 tokens), against
// the merges into the slab and the GEMM that reads it.  us.  Fused: rounds of tasks over the CUs times their K steps, whose
// expert chunks grow with E and are shared by up to eight row chunks; extra_us is added.  Slab: the bytes of the merges and of
// the GEMM.  The first two segments of every sequence share their merged values: one of them is not stored, and read
// from the cache in part.  Fitted to both forms of 600 layers each of 64- and 128-token segments (1 .. 120 sequences of 2 .. 240
// segments, 2 .. 16 experts, d = 768 .. 2560, d_ff = 704 .. 6144): off by 9 and 8 % (rms).  The margins keep out what is not
// clearly faster: 0.94 with 64- and 0.90 with 128-token segments, 38 of 3540 contractions take 3 % longer than through the slab,
// 1.18 at worst (0.90 for both: 29, but 0.5 % of the gain is lost); with few segments the merges run at the memory's rate and
// rounds of tasks are unevenly filled: 0.76.  Time of the slab's that is left,
// many segments, T = 64: gate/up 0.56, down 0.72, dA 0.61, dX 0.78; T = 128: 0.95, 0.99, 0.96, 1.00; few segments, T = 64:
// 0.88, 1.00, 0.95, 1.00 (T = 128 0.98 for gate/up, 1.25 at worst: the slab).  us of slab and fused: gate/up of 82 segments of
// 64, 7 experts of 1792 x 4160 1280 and 650; dX of 3 segments, 14 of 1792 x 5632 230 and 650; a backward pass of 16 sequences of two
// 128-token segments, 4 of 2048 x 5632 1901 and 1997.  One expert always takes the slab: its segments share their merged values.
// Layers of fewer parameters than measured stay on the slab with 128-token segments, where the two forms are close.
constexpr long kFusedLeastD = 500000;

double slab_us(const Dims &m, int mats)
{
    const long distinct = m.N > 1 ? m.S - m.B : m.S;
    return 15.0 + mats * (6.9 + 2e-6 * m.D * (0.215 * distinct + (m.T > 64 ? 0.215 : 0.172) * m.S + 0.165 * m.E));
}

bool fused_pays(const Dims &m, int N, int K, int mats, int nsrc, double extra_us = 0.0)
{
    const bool few = k::merge_is_few(m.S, m.E);
    if (m.E < 2 || (m.T > 64 && (few || m.D < kFusedLeastD))) return false;
    const long cus = gemm2::cu_count(), chunks = (m.tokens + fmg::kRows8 - 1) / fmg::kRows8;
    const long tasks = chunks * (N / fmg::BN) * (mats / nsrc), rounds = ((tasks + 7) / 8 + cus / 8 - 1) / (cus / 8);
    const double fused = 8.3 + extra_us + (double)rounds * nsrc * (K / fmg::BK) * (1.17 + m.E * (0.038 + 0.031 / (chunks < 8 ? chunks : 8)));
    return fused < (few ? 0.76 : m.T > 64 ? 0.90 : 0.94) * slab_us(m, mats);
}

// The same on the four-wave kernel, for stacks of 4 GiB and more, which the eight-wave kernel does not take.  Supertasks of 8
// row chunks by 4 column blocks, one to an XCD at a time; with fewer than four row chunks hardly any expert chunk is shared.
// A K step of K-slow stacks takes 2.3 us with 8 experts and 2.45 with 16, of K-contiguous ones (dA, dX) 2.2 and 3.5.
// ms of slab and fused, 8192 tokens in segments of 64: gate/up, down of 16 experts of 8192 x 16384 28.5, 14.2 and 20.4, 10.2
// (2048 tokens 8.3, 4.1 and 10.2, 5.1), dA + dX 42 and 44; backward pass of 16384 tokens, 8 of 16384 x 16384 378 and 318.
bool fused_pays_four(const Dims &m, int N, int K, int mats, bool k_slow)
{
    const long chunks = (m.tokens + fmg::kRows8 - 1) / fmg::kRows8, super = (chunks + 7) / 8 * ((N / fmg::BN + 3) / 4);
    const double step = k_slow ? 2.15 + 0.019 * m.E : 0.9 + 0.163 * m.E;
    const double fused = mats * (10.0 + (double)((super + 7) / 8) * (K / fmg::BK) * step);
    return m.T <= 64 && m.E >= 2 && m.E <= 16 && chunks >= 4 && fused < 0.90 * slab_us(m, mats);
}

// The contractions of the layer have N and K in {d, d_ff}: parameters of the two products, for the shape conditions alone.
fmg::Params fused_shape(const Dims &m, bool n_is_dff)
{
    const int N = n_is_dff ? m.dff : m.d, K = n_is_dff ? m.d : m.dff;
    return fused_params(m, nullptr, nullptr, K, nullptr, nullptr, N, nullptr, N, K, nullptr, N);
}

// Whether the eight-wave kernel takes every contraction of the layer.
bool eight_waves(const Dims &m)
{
    const fmg::Params a = fused_shape(m, true), b = fused_shape(m, false);
    return m.tokens <= 0x7fffffffL && ((fmg::fits8<64>(a) && fmg::fits8<64>(b)) || (fmg::fits8<128>(a) && fmg::fits8<128>(b)));
}

// keep_gu: the caller keeps G and U (or, in a backward pass, they are recomputed into bf16 planes).  Without, the fused kernel
// writes them in fp32 and the activation is a pass of its own, 16 bytes an element more than the epilogue of the slab
// pipeline moves.
Fused use_fused(const Dims &m, bool keep_gu)
{
    const Fused none = {false, false, false, false}, all = {true, true, true, true};
    const int mode = fused_mode();
    if (mode == 0 || m.tokens > 0x7fffffffL) return none;
    const bool fits = k::fused_fits(fused_shape(m, true)) && k::fused_fits(fused_shape(m, false));
    if (!fits || mode >= 2) return fits ? all : none;
    // longer segments, more experts and stacks of 4 GiB and more run on the four-wave kernel, which does not write fp32 planes
    if (!eight_waves(m))
        return {keep_gu && fused_pays_four(m, m.dff, m.d, 2, true), fused_pays_four(m, m.d, m.dff, 1, true),
                fused_pays_four(m, m.dff, m.d, 1, false), fused_pays_four(m, m.d, m.dff, 2, false)};
    const bool gate_up = fused_pays(m, m.dff, m.d, 2, 1, keep_gu ? 0.0 : 3.4e-6 * m.tokens * m.dff);
    return {gate_up, fused_pays(m, m.d, m.dff, 1, 1), fused_pays(m, m.dff, m.d, 1, 1),
            fused_pays(m, m.d, m.dff, 2, 2)};
}

// Whether the backward keeps the per-segment weight gradients on chip as well (fsg_kernel), for
// shapes that kernel takes.
bool use_fused_dw() { return fused_mode() == 3; }

// One fused contraction: C = sum over sources of A_q * Wbar_q(segment), merged on chip.
hipError_t fused_gemm(hipStream_t st, const Dims &m, int cls, const fmg::Params &p, int nsrc, bool w_nc)
{
    const double D = (double)p.N * p.K;
    prof::Range r(st, cls, nsrc * (2.0 * p.tokens * D + 4.0 * m.S * m.E * D),
                  2.0 * (nsrc * ((double)m.E * D + (double)p.tokens * p.K) + (double)p.tokens * p.N));
    return k::launch_fused(st, p, nsrc, w_nc);
}

// Gate and up projections of all tokens, merged on chip; in fp32 (G and U are then of that type) or rounded.
hipError_t fused_gate_up(hipStream_t st, const Dims &m, const bf *X, const bf *Wg, const bf *Wu, const float *w, bf *G, bf *U,
                         bool f32)
{
    fmg::Params p = fused_params(m, X, nullptr, m.d, Wg, Wu, m.dff, w, m.dff, m.d, G, m.dff);
    p.C2 = U;
    const double D = (double)m.D;
    prof::Range r(st, prof::kFusedGU, 2.0 * (2.0 * m.tokens * D + 4.0 * m.S * m.E * D),
                  2.0 * (2.0 * m.E * D + (double)m.tokens * m.d + (f32 ? 4.0 : 2.0) * m.tokens * m.dff));
    return f32 ? k::launch_fused_pair_f32(st, p) : k::launch_fused_pair(st, p);
}

// Largest multiple of `gran` that is <= limit and <= full, at least gran.
int block_width(size_t budget, size_t bytes_per_unit, int full, int gran)
{
    long wdt = (long)(budget / bytes_per_unit) / gran * gran;
    if (wdt < gran) wdt = gran;
    if (wdt > full) wdt = full;
    return (int)wdt;
}

struct Plan {
    int Sc;        // segments per chunk (limits of the merge / scatter kernels)
    int gran_f;    // granularity of d_ff blocks
    int gran_d;    // granularity of d blocks
    int nf_fwd, jf_fwd, nf_bwd, kf_bwd;
    size_t act;        // bytes of one [chunk tokens, d_ff] bf16 buffer
    size_t slab_fwd;   // bytes of the forward slab region
    size_t slab_bwd;   // bytes of the backward slab region
    size_t partials;   // bytes of the router-weight partial sums
    int prow, pcol;
};

Plan make_plan(const Dims &m)
{
    Plan p;
    const int cap = (m.E <= 32) ? 256 : 128;  // routing-weight operand tables of the merge kernel (LDS)
    p.Sc = m.S < cap ? m.S : cap;
    p.gran_f = (m.dff % 256 == 0) ? 256 : (m.dff % 128 == 0) ? 128 : 64;
    p.gran_d = (m.d % 256 == 0) ? 256 : (m.d % 128 == 0) ? 128 : 64;
    const size_t budget = slab_budget_bytes();
    const size_t S = (size_t)p.Sc;
    p.nf_fwd = block_width(budget, S * m.d * 2 * 2, m.dff, p.gran_f);
    p.jf_fwd = block_width(budget, S * m.dff * 2, m.d, p.gran_d);
    p.nf_bwd = block_width(budget, S * m.d * 2 * 4, m.dff, p.gran_f);
    p.kf_bwd = block_width(budget, S * m.dff * 2 * 2, m.d, p.gran_d);
    p.act = align_up((size_t)p.Sc * m.T * m.dff * 2, 256);
    const size_t gu = S * m.d * p.nf_fwd * 2 * 2, dn = S * m.dff * p.jf_fwd * 2;
    p.slab_fwd = align_up(gu > dn ? gu : dn, 256);
    const size_t ph = S * m.d * p.nf_bwd * 2 * 4, dx = S * m.dff * p.kf_bwd * 2 * 2;
    const size_t re = S * m.d * p.nf_bwd * 2 * 2;  // gate/up slabs when G, U are recomputed
    size_t b = ph > dx ? ph : dx;
    if (re > b) b = re;
    p.slab_bwd = align_up(b, 256);
    k::scatter_partial_dims(p.Sc, m.E, &p.prow, &p.pcol);
    p.partials = align_up((size_t)k::scatter_grid() * p.prow * p.pcol * sizeof(float), 256);
    return p;
}

#define LORY_TRY(expr)                                   \
    do {                                                 \
        if ((expr) != hipSuccess) return LORY_ERR_DEVICE; \
    } while (0)

Rect rect(long D, int pitch, int r0, int nr, int c0, int nc)
{
    Rect rc;
    rc.expert_stride = D;
    rc.pitch = pitch;
    rc.r0 = r0;
    rc.nr = nr;
    rc.c0 = c0;
    rc.nc = nc;
    return rc;
}

// The map of segments that share their merged values (MergeParams::seg_map), in memory that lies unused between two
// places while the slab is written and read; NULL where there is too little.
constexpr size_t kMapElems = ms::kMapSegments * sizeof(int32_t) / sizeof(bf) + 128;   // with the rounding to 256 bytes

int32_t *map_place(int S, void *from, void *to)
{
    const size_t a = align_up((size_t)from, 256);
    return S > 1 && S <= ms::kMapSegments && a + ms::kMapSegments * sizeof(int32_t) <= (size_t)to ? (int32_t *)a : nullptr;
}

// Scratch for a cut last round of tiles: what lies unused between two places of the workspace while the GEMM runs.
// Only where the transient slab holds the whole matrix, and the same scratch whether the merged parameters are saved or
// not: the sums of the two modes are then added in the same order.
void set_tail(Params &p, bool whole, void *from, void *to)
{
    if (!whole) return;
    const size_t a = align_up((size_t)from, 256), b = (size_t)to;
    p.tail = b > a ? (float *)a : nullptr;
    p.tail_floats = b > a ? (b - a) / sizeof(float) : 0;
}

// Sizes and scratch of the token GEMMs whose last round of tiles may be cut, for S segments with the slab at `slab`.
Params down_gemm(const Dims &m, const Plan &pl, bool whole, int S, int jf, bf *slab)
{
    Params p = {};
    p.M = m.T; p.N = jf; p.K = m.dff; p.batches = S;
    set_tail(p, whole, slab + (size_t)S * m.dff * jf + kMapElems, (char *)slab + pl.slab_fwd);
    return p;
}

Params da_gemm(const Dims &m, const Plan &pl, int S, int nf, bf *slab)
{
    Params p = {};
    p.M = m.T; p.N = nf; p.K = m.d; p.batches = S;
    set_tail(p, nf == m.dff, slab + (size_t)S * m.d * nf + kMapElems, (char *)slab + pl.slab_bwd);
    return p;
}

Params dx_gemm(const Dims &m, const Plan &pl, int S, int kf, bf *slab)
{
    Params p = {};
    p.M = m.T; p.N = kf; p.K = m.dff; p.batches = S;
    set_tail(p, kf == m.d, slab + (size_t)2 * S * m.dff * kf + kMapElems, (char *)slab + pl.slab_bwd);
    return p;
}

double gemm_flops(const Params &p, int nset, int nsrc)
{
    return 2.0 * p.batches * p.M * p.N * p.K * nset * nsrc;
}

// Merges of `count` matrices with the same rectangle, each into a slab of its own; of more than one only where few
// segments are merged (k::merge_is_few).
hipError_t merge(hipStream_t st, const float *w, int S, int E, const bf *const *stack, int count, const Rect &rc, bf *const *slab,
                 int32_t *seg_map)
{
    const double n = (double)rc.nr * rc.nc;
    int rec;
    {
        prof::Range r(st, prof::kMerge, 2.0 * S * E * n * count, 2.0 * n * (E + S) * count);
        rec = r.index();
        hipError_t e;
        if (k::merge_is_few(S, E)) {
            ms::MergeFewParams p = {};
            p.w = w;
            p.S = S;
            p.E = E;
            for (int x = 0; x < count; ++x) {
                p.stack[x] = stack[x];
                p.slab[x] = slab[x];
            }
            p.rc = rc;
            p.seg_stride = (long)rc.nr * rc.nc;
            p.seg_map = seg_map;
            e = k::launch_merge_few(st, p, count);
        } else {
            if (count != 1) return hipErrorInvalidValue;
            MergeParams p;
            p.w = w;
            p.S = S;
            p.E = E;
            p.stack = stack[0];
            p.rc = rc;
            p.slab = slab[0];
            p.seg_stride = (long)rc.nr * rc.nc;
            p.seg_map = seg_map;
            e = k::launch_merge(st, p);
        }
        if (e != hipSuccess) return e;
    }
    prof::shared_segments(st, rec, seg_map, S, 2.0 * n * count);
    return hipSuccess;
}

hipError_t merge(hipStream_t st, const float *w, int S, int E, const bf *stack, const Rect &rc, bf *slab,
                 int32_t *seg_map = nullptr)
{
    return merge(st, w, S, E, &stack, 1, rc, &slab, seg_map);
}

// Gate/up projections of one d_ff column block for a chunk of segments.
hipError_t gate_up_block(hipStream_t st, const Dims &m, int S, const bf *X, const float *w, const bf *Wg,
                         const bf *Wu, int n0, int nf, bf *slab, bf *G, bf *U, bf *Act, bf *slab_up = nullptr,
                         int32_t *seg_map = nullptr)
{
    bf *sg = slab, *su = slab_up ? slab_up : slab + (size_t)S * m.d * nf;
    const Rect rc = rect(m.D, m.dff, 0, m.d, n0, nf);
    hipError_t e;
    if ((e = merge(st, w, S, m.E, Wg, rc, sg, seg_map)) != hipSuccess) return e;
    if ((e = merge(st, w, S, m.E, Wu, rc, su, seg_map)) != hipSuccess) return e;
    Params p = {};
    p.A[0] = X; p.a_batch[0] = (long)m.T * m.d; p.lda[0] = m.d;
    p.B[0] = sg; p.b_batch[0] = (long)m.d * nf; p.ldb[0] = nf;
    p.B[1] = su; p.b_batch[1] = (long)m.d * nf; p.ldb[1] = nf;
    p.b_map = seg_map;
    p.M = m.T; p.N = nf; p.K = m.d; p.batches = S;
    // With G and U saved anyway, the activation A = silu(G) * U is cheaper as a streaming pass
    // over them than as a third output plane of the GEMM epilogue; without saved G, U it is
    // computed in the epilogue from the fp32 accumulators.
    const bool split = (G != nullptr && Act != nullptr);
    EpiGU epi = {G, U, split ? nullptr : Act, m.T, m.dff, n0};
    const double out_elems = (double)S * m.T * nf * ((G ? 2 : 0) + ((Act && !split) ? 1 : 0));
    int rec;
    {
        prof::Range r(st, prof::kGemmGU, gemm_flops(p, 2, 1),
                      2.0 * ((double)S * m.T * m.d + 2.0 * S * m.d * nf + out_elems));
        rec = r.index();
        if ((e = k::launch_gu(st, p, epi)) != hipSuccess) return e;
    }
    prof::shared_segments(st, rec, seg_map, S, 4.0 * m.d * nf);
    if (split) {
        prof::Range r(st, prof::kSwigluFwd, 4.0 * S * m.T * nf, 2.0 * 3.0 * S * m.T * nf);
        return k::launch_swiglu_fwd(st, G, U, Act, (long)S * m.T, m.dff, n0, nf);
    }
    return hipSuccess;
}

}  // namespace

int set_fused_mode(int mode)
{
    if (mode < 0 || mode > 3) return LORY_ERR_SHAPE;
    g_fused_mode = mode;
    return LORY_OK;
}

int set_slab_budget(size_t bytes)
{
    if (bytes < ((size_t)64 << 10)) return LORY_ERR_SHAPE;
    g_slab_budget = bytes;
    return LORY_OK;
}

size_t bf16_merged_save_bytes(const Dims &m)
{
    const Plan p = make_plan(m);
    if (m.S > p.Sc) return 0;  // more segments than one merge launch handles
    return (size_t)3 * m.S * m.D * 2;
}

// How the fused gate and up projections leave G and U in the workspace of a forward pass whose caller does not keep them:
// in fp32 where that fits the slab, so that the activation rounds once as in the slab pipeline's epilogue.  Otherwise the call
// takes the slab, at every token count, and asks for no more workspace than it; only where the merge inside the GEMM is asked
// for (modes 2 and 3) the planes are rounded.  Error of Y against 64 bits, 1e-3, 11 segments of 64, 8 experts of 512 x 1408: slab
// 3.714, fp32 planes 3.713, rounded planes 4.46.
enum class Planes { kNone, kF32, kBf16 };

Planes gate_up_planes(const Dims &m, const Plan &p, bool explicitly)
{
    if (eight_waves(m) && 4 * p.act <= p.slab_fwd) return Planes::kF32;
    return explicitly ? Planes::kBf16 : Planes::kNone;
}

size_t bf16_workspace_bytes(const Dims &m, int pass)
{
    const Plan p = make_plan(m);
    if (pass == LORY_PASS_FWD) {
        // rounded G and U of all tokens when the caller does not keep them
        const bool explicitly = fused_mode() > 1;
        const size_t gu = explicitly && use_fused(m, false).gate_up && gate_up_planes(m, p, explicitly) == Planes::kBf16 ? 2 * p.act : 0;
        return p.act + (p.slab_fwd > gu ? p.slab_fwd : gu);
    }
    // dG, dU, Act, recomputed G and U, slabs, router-weight partial sums
    return 5 * p.act + p.slab_bwd + p.partials;
}

LayerForm bf16_layer_form(const Dims &m)
{
    const Plan pl = make_plan(m);
    bf *slab = (bf *)256;   // nothing is launched
    const int S = pl.Sc, jf = pl.jf_fwd, nf = pl.nf_bwd, kf = pl.kf_bwd;
    auto form = [](const Params &p, int nsrc) -> TileForm {
        const gemm2::Form f = gemm2::tile_form(p, 256, nsrc);
        const long tiles = (long)p.batches * ((p.M + f.rows - 1) / f.rows) * ((p.N + 255) / 256);
        return {f.rows, f.pieces, (int)(tiles / gemm2::cu_count())};
    };
    return {form(down_gemm(m, pl, jf == m.d, S, jf, slab), 1), form(da_gemm(m, pl, S, nf, slab), 1), form(dx_gemm(m, pl, S, kf, slab), 2)};
}

int bf16_ffn_fwd(const Dims &m, const void *Xv, const float *w, const void *Wgv, const void *Wuv,
                 const void *Wdv, void *Yv, void *Gv, void *Uv, void *Wbarv, void *ws, hipStream_t st)
{
    Plan pl = make_plan(m);
    const bool whole_d = pl.jf_fwd == m.d;
    bf *Wbar = (bf *)Wbarv;  // [Wg_bar | Wu_bar | Wd_bar], each [S][rows][cols]; doubles as the slab
    if (Wbar) {
        pl.nf_fwd = m.dff;
        pl.jf_fwd = m.d;
    }
    const bf *X = (const bf *)Xv, *Wg = (const bf *)Wgv, *Wu = (const bf *)Wuv, *Wd = (const bf *)Wdv;
    bf *Y = (bf *)Yv, *G = (bf *)Gv, *U = (bf *)Uv;
    bf *Act = (bf *)ws;
    bf *slab = (bf *)((char *)ws + pl.act);
    const long TD = (long)m.T * m.d, TF = (long)m.T * m.dff;

    Fused fused = Wbar || m.S > pl.Sc ? Fused{} : use_fused(m, G != nullptr);
    const Planes planes = G ? Planes::kBf16 : gate_up_planes(m, pl, fused_mode() > 1);
    if (planes == Planes::kNone) fused.gate_up = false;
    if (fused.gate_up) {
        // merged parameters never leave the chip: fused contractions and one SwiGLU pass
        const double elements = (double)m.tokens * m.dff;
        if (planes == Planes::kF32) {
            float *Gf = (float *)slab, *Uf = (float *)((char *)slab + 2 * pl.act);
            LORY_TRY(fused_gate_up(st, m, X, Wg, Wu, w, (bf *)Gf, (bf *)Uf, true));
            prof::Range r(st, prof::kSwigluFwd, 4.0 * elements, 10.0 * elements);
            LORY_TRY(k::launch_swiglu_fwd_f32(st, Gf, Uf, Act, m.tokens * m.dff));
        } else {
            bf *Gf = G ? G : slab, *Uf = U ? U : (bf *)((char *)slab + pl.act);
            LORY_TRY(fused_gate_up(st, m, X, Wg, Wu, w, Gf, Uf, false));
            prof::Range r(st, prof::kSwigluFwd, 4.0 * elements, 2.0 * 3.0 * elements);
            LORY_TRY(k::launch_swiglu_fwd(st, Gf, Uf, Act, m.tokens, m.dff, 0, m.dff));
        }
    }

    for (int s0 = 0; s0 < m.S; s0 += pl.Sc) {
        const int S = (m.S - s0 < pl.Sc) ? (m.S - s0) : pl.Sc;
        const float *wc = w + (size_t)s0 * m.E;
        const bf *Xc = X + (size_t)s0 * TD;
        bf *Gc = G ? G + (size_t)s0 * TF : nullptr;
        bf *Uc = U ? U + (size_t)s0 * TF : nullptr;
        // Y is written by the down projection alone: until then it holds the map (unless it is X as well)
        const char *y0 = (const char *)(Y + (size_t)s0 * TD), *y1 = y0 + sizeof(bf) * S * TD;
        const char *x0 = (const char *)X, *x1 = x0 + sizeof(bf) * m.tokens * m.d;
        int32_t *map_gu = (y1 <= x0 || x1 <= y0) ? map_place(S, (void *)y0, (void *)y1) : nullptr;
        // gate / up projections + SwiGLU, one d_ff column block at a time
        for (int n0 = 0; !fused.gate_up && n0 < m.dff; n0 += pl.nf_fwd) {
            const int nf = (m.dff - n0 < pl.nf_fwd) ? (m.dff - n0) : pl.nf_fwd;
            if (Wbar)
                LORY_TRY(gate_up_block(st, m, S, Xc, wc, Wg, Wu, n0, nf, Wbar, Gc, Uc, Act,
                                       Wbar + (size_t)m.S * m.D));
            else
                LORY_TRY(gate_up_block(st, m, S, Xc, wc, Wg, Wu, n0, nf, slab, Gc, Uc, Act, nullptr, map_gu));
        }
        if (fused.down) {
            LORY_TRY(fused_gemm(st, m, prof::kFusedDown,
                                fused_params(m, Act, nullptr, m.dff, Wd, nullptr, m.d, w, m.d, m.dff, Y, m.d), 1, true));
            continue;
        }
        // down projection, one block of output columns at a time
        for (int j0 = 0; j0 < m.d; j0 += pl.jf_fwd) {
            const int jf = (m.d - j0 < pl.jf_fwd) ? (m.d - j0) : pl.jf_fwd;
            bf *sd = Wbar ? Wbar + (size_t)2 * m.S * m.D : slab;
            bf *past = slab + (size_t)S * m.dff * jf;
            int32_t *map = Wbar ? nullptr : map_place(S, past, (char *)slab + pl.slab_fwd);
            LORY_TRY(merge(st, wc, S, m.E, Wd, rect(m.D, m.d, 0, m.dff, j0, jf), sd, map));
            Params p = down_gemm(m, pl, whole_d, S, jf, slab);
            p.b_map = map;
            p.A[0] = Act; p.a_batch[0] = TF; p.lda[0] = m.dff;
            p.B[0] = sd; p.b_batch[0] = (long)m.dff * jf; p.ldb[0] = jf;
            EpiStore epi = {Y + (size_t)s0 * TD + j0, TD, m.d};
            int rec;
            {
                prof::Range r(st, prof::kGemmDown, gemm_flops(p, 1, 1),
                              2.0 * ((double)S * TF + (double)S * m.dff * jf + (double)S * m.T * jf));
                rec = r.index();
                LORY_TRY(k::launch_down(st, p, epi));
            }
            prof::shared_segments(st, rec, map, S, 2.0 * m.dff * jf);
        }
    }
    return LORY_OK;
}

// Merged parameters of all m.S segments, materialised as [Wg_bar | Wu_bar | Wd_bar], each
// [S][rows][cols] (the layout of Wbar_save).
int bf16_merge_all(const Dims &m, const float *w, const void *Wgv, const void *Wuv, const void *Wdv,
                   void *Wbarv, hipStream_t st)
{
    const Plan pl = make_plan(m);
    const bf *stacks[3] = {(const bf *)Wgv, (const bf *)Wuv, (const bf *)Wdv};
    const Rect all = rect(m.D, (int)m.D, 0, 1, 0, (int)m.D);   // whole matrices lie in one piece
    bf *out = (bf *)Wbarv;
    for (int s0 = 0; s0 < m.S; s0 += pl.Sc) {
        const int S = (m.S - s0 < pl.Sc) ? (m.S - s0) : pl.Sc;
        bf *slabs[3] = {out + (size_t)s0 * m.D, out + ((size_t)m.S + s0) * m.D, out + ((size_t)2 * m.S + s0) * m.D};
        const float *ws = w + (size_t)s0 * m.E;
        if (k::merge_is_few(S, m.E)) {
            LORY_TRY(merge(st, ws, S, m.E, stacks, 3, all, slabs, nullptr));
            continue;
        }
        for (int x = 0; x < 3; ++x) LORY_TRY(merge(st, ws, S, m.E, stacks[x], all, slabs[x]));
    }
    return LORY_OK;
}

namespace {

void *const kNoWorkspace = (void *)256;   // stands for one where a call is planned and not launched

// Tile height and K slices of one projection of the dense FFN.
struct DenseSplit {
    int rows;
    int ks;      // 0: not split, launch_rows picks the tile (of `rows`)
    double us;   // estimated time
};

// Estimated time, us, of a projection of up to 128 rows (decode steps, short blocks): it streams the weights, so
// a round of tiles over the CUs takes its K steps at the latency of the ring, or at the rate the chip reads memory
// when enough CUs take part (0.7 us for 16 KB on each of 256: 6 TB/s), and a nearly empty last round costs its steps
// all the same.  Fitted to 25 forms each of 41 projections (1 .. 16 sequences of 1 .. 128 tokens, d = 256 .. 2560) whose
// weights are read from memory, as between the layers of a model: what it picks is 0.25 us slower than the fastest
// form on average.
double stream_us(int rows, long tiles, int steps, int cus)
{
    const double lat = rows == 64 ? 0.52 : 0.64, mem = (rows == 64 ? 0.70 : 0.66) / cus;
    auto round = [&](long n) { return steps * (mem * n > lat ? mem * n : lat) + 1.2; };
    return (rows == 64 ? 2.5 : 4.0) + (tiles / cus) * round(cus) + (tiles % cus ? round(tiles % cus) : 0.0);
}

// M rows per sequence, N columns per operand set, nset operand sets, the row operand in `terms` bf16 terms (unsplit: one
// source each; split: rows of their own, whose sums are added with those of the slices).  A few dozen rows against one
// weight matrix per sequence leave CUs without a tile or the last round of tiles nearly empty, and the pass is bound by
// how many CUs stream the weights, so the contraction is cut into slices; what they cost is a launch that adds their
// fp32 partial sums (4.5 us with the gap before it) and those sums (written once, read once: 0.6 us a million where a
// tile holds all rows, 2 beyond).  Blocks of more rows than a tile are cut until the tiles fill the chip once (beyond
// 128 rows by step_us, with six steps for the fill of the ring and the epilogue).  max_floats bounds the partial sums.
// us per call with weights from memory, one round of tiles at most and 3 us for the sums -> this: 12 sequences at
// d = 2560, d_ff = 6144 224 -> 208 (207 on the vector ALUs), 6 at d = 2048, d_ff = 5632 100 -> 90.
DenseSplit dense_split(const Dims &m, int M, int N, int K, int nset, int terms, size_t max_floats)
{
    const int cus = gemm2::cu_count(), bns = 256 / nset, steps = K / gemm2::BK;
    auto tiles_of = [&](int r, int rows) { return (long)m.B * ((r + rows - 1) / rows) * ((N + bns - 1) / bns); };
    auto rounds_us = [&](int rows, long tiles, int k) {
        return gemm2::step_us(rows) * ((double)((tiles + cus - 1) / cus) * k + 6);
    };
    Params p = {};
    p.M = M; p.N = N; p.batches = m.B;
    const int whole = gemm2::tile_rows(p, bns);
    const long tiles1 = tiles_of(M, whole);
    DenseSplit best = {whole, 0, (M <= 128 && whole <= 128) ? stream_us(whole, tiles1, terms * steps, cus)
                                                            : rounds_us(whole, tiles1, terms * steps)};
    for (int rows = 64; rows <= 128 && K <= gemm2::kMaxCutK; rows += rows) {
        const long tiles = tiles_of(terms * M, rows);
        const bool few = terms * M <= 128, one = terms * M <= rows;
        for (int ks = 1; ks <= steps / 4 && (one || tiles * ks <= cus); ++ks) {
            const double parts = (double)ks * nset * terms * m.B * M * N;
            if (parts > (double)max_floats) break;
            const int k = (steps + ks - 1) / ks;
            const double t = (few ? stream_us(rows, tiles * ks, k, cus) : rounds_us(rows, tiles, k)) + parts * (one ? 6e-7 : 2e-6) + 4.5;
            if (t < best.us) best = {rows, ks, t};
        }
    }
    return best;
}

// Rows of the dense FFN are walked in blocks of `rows` per sequence (all of them unless the scratch is too small).
struct DensePlan {
    int terms;           // bf16 terms of the activation
    int rows;
    size_t act;          // bytes of a block's activation
    size_t floats;       // bound on the partial sums of split contractions
    bool fixed;          // the scratch is
    DenseSplit gate_up(const Dims &m, int r) const { return dense_split(m, r, m.dff, m.d, 2, 1, floats); }
    DenseSplit down(const Dims &m, int r) const { return dense_split(m, r, m.d, m.dff, 1, terms, floats); }
    // The down projection where it is not split as a whole: its last round of tiles may be, unless the call is held to a
    // fixed scratch.
    Params down_params(const Dims &m, int r, void *ws, size_t ws_bytes) const
    {
        Params p = {};
        p.M = r; p.N = m.d; p.K = m.dff; p.batches = m.B;
        if (!fixed && ws_bytes > act) {
            p.tail = (float *)((char *)ws + act);
            p.tail_floats = (ws_bytes - act) / sizeof(float);
        }
        return p;
    }
    size_t parts(const Dims &m, int r) const   // floats that a block of r rows uses
    {
        const DenseSplit g = gate_up(m, r), w = down(m, r);
        const size_t a = g.ks ? (size_t)g.ks * 2 * m.B * r * m.dff : 0;
        const size_t b = w.ks ? (size_t)w.ks * terms * m.B * r * m.d : 0;
        return a > b ? a : b;
    }
    // K slices of the streaming gate/up projections, 0: the ring GEMM.  Where the latter is not cut it forms the activation
    // in its epilogue, which neither the sums through memory nor the launch that reads them can match: 4 sequences of 64
    // rows at d = 2048, d_ff = 5632 73 us a call, streamed 82.  The sums stay within the ring GEMM's.
    int stream_gu(const Dims &m, int r) const
    {
        const DenseSplit g = gate_up(m, r);
        return g.ks ? k::dense_stream_gu_slices(m.B, r, m.d, m.dff, parts(m, r), g.us) : 0;
    }
};

DensePlan dense_plan(const Dims &m, const DenseScratch &scratch)
{
    DensePlan p;
    p.fixed = scratch.fixed;
    // Blocks of 64 k tokens (prefill) round the activation to bf16 like the training forward; every other
    // number of tokens, decode steps among them, keeps it in fp32 precision.
    p.terms = m.L % 64 == 0 ? 1 : 2;
    const size_t per_row = (size_t)m.B * m.dff * 2 * p.terms;
    p.rows = m.L;
    if (scratch.fixed && per_row * m.L > scratch.bytes) {
        size_t r = scratch.bytes / per_row;
        if (r < 1) r = 1;
        // blocks of equal size, in whole tiles where one fits
        const size_t n = ((size_t)m.L + r - 1) / r, even = ((size_t)m.L + n - 1) / n;
        p.rows = (int)(r >= 64 ? (even + 63) / 64 * 64 <= r ? (even + 63) / 64 * 64 : r / 64 * 64 : r);
    }
    p.act = align_up(per_row * p.rows, 256);
    p.floats = scratch.bytes > p.act ? (scratch.bytes - p.act) / 256 * 256 / sizeof(float) : 0;
    return p;
}

}  // namespace

size_t bf16_dense_workspace_bytes(const Dims &m, const DenseScratch &scratch)
{
    const DensePlan p = dense_plan(m, scratch);
    const int last = m.L % p.rows;
    size_t parts = p.parts(m, p.rows);
    if (last) {
        const size_t q = p.parts(m, last);
        if (q > parts) parts = q;
    }
    return p.act + align_up(parts * sizeof(float), 256);
}

// Scratch of a cut last round of the down projection, for calls that are not held to a fixed scratch.
size_t bf16_dense_tail_bytes(const Dims &m, const DenseScratch &scratch)
{
    const DensePlan p = dense_plan(m, scratch);
    if (p.down(m, m.L).ks) return 0;
    const Params q = p.down_params(m, m.L, kNoWorkspace, (size_t)1 << 60);
    return p.act + gemm2::tail_floats(q, gemm2::tile_form(q, 256, p.terms), 256) * sizeof(float);
}

DenseForm bf16_dense_form(const Dims &m, const DenseScratch &scratch, size_t ws_bytes, const DenseStream &sp)
{
    const DensePlan p = dense_plan(m, scratch);
    if (sp.gu) return {m.L, 2, 0, 0, 0, 0, 0, sp};
    const DenseSplit g = p.gate_up(m, p.rows), d = p.down(m, p.rows);
    const int ks = p.stream_gu(m, p.rows);
    DenseForm f = {p.rows, p.terms, ks ? 0 : g.rows, ks ? 0 : g.ks, d.rows, d.ks, 0, {ks, 0}};
    if (!d.ks) {
        const gemm2::Form t = gemm2::tile_form(p.down_params(m, p.rows, kNoWorkspace, ws_bytes), 256, p.terms);
        f.down_tile = t.rows;
        f.down_pieces = t.pieces;
    }
    return f;
}

// Every block of up to 10 rows streams.  So do 11 .. 16, unless the ring GEMM would form the activation in the epilogue of
// an uncut gate/up whose last round of tiles uses half the CUs or more, and has the K steps or the rounds to pay for its
// fill: from 13 rows on at d = 1024 and wider, from 11 on with a second round there or a third below.  us, streamed and ring
// GEMM.  16 rows: 4 sequences at d = 1216, d_ff = 4992 (156 tiles) 41.1 and 37.4, 8 at 1536, 4096 (256) 70.8 and 65.8,
// 3 at 2048, 5632 (132) 56.1 and 54.7, 48 at 768, 2048 (768) 109 and 100; 8 at 768, 6144 (384) 54.3 and 57.6, 8 at 768, 2048
// (128) 25.1 and 28.1.  12 rows: 10 at 1216, 4992 (390) 81.3 and 75.9, 48 there (1872) 333 and 310, 20 at 1024, 2816 (440)
// 74.6 and 72.0; in one round 1.00 of the ring GEMM's time on average, 0.92 .. 1.04.  8 rows: 0.88 .. 1.02, 0.96 on average.
DenseStream bf16_dense_stream_plan(const Dims &m, size_t ws_bytes, const DenseScratch &scratch)
{
    if (m.L > 10 && m.L <= 16) {
        const DensePlan p = dense_plan(m, scratch);
        const DenseSplit g = p.gate_up(m, p.rows);
        const long cus = gemm2::cu_count(), tiles = (long)m.B * ((p.rows + g.rows - 1) / g.rows) * ((m.dff + 127) / 128);
        const long rounds = (tiles + cus - 1) / cus;
        const bool pays = m.d >= 1024 ? m.L > 12 || rounds >= 2 : rounds >= 3;
        if (!g.ks && pays && 2 * tiles >= rounds * cus) return {0, 0};
    }
    return k::dense_stream_plan(m.B, m.L, m.d, m.dff, ws_bytes / sizeof(float));
}

// Decode steps and blocks of at most 16 rows: two streaming projections, the gate/up sums between them in the scratch.
int bf16_dense_stream(const Dims &m, const DenseStream &sp, const void *X, const void *Wbarv, void *Yv, void *scratch, hipStream_t st)
{
    const bf *Wbar = (const bf *)Wbarv;
    bf *Y = (bf *)Yv;
    float *ws = (float *)scratch, *parts = ws + (size_t)sp.gu * 2 * m.B * m.L * m.dff;
    stream::Params p = {};
    p.M = m.L;
    p.w_batch = m.D;
    {
        prof::Range r(st, prof::kGemmGU, 4.0 * m.tokens * m.D, 2.0 * (m.tokens * (double)m.d + 2.0 * m.B * m.D));
        p.K = m.d; p.N = m.dff; p.ks = sp.gu;
        p.W[0] = Wbar; p.W[1] = Wbar + (size_t)m.B * m.D;
        p.x = (const bf *)X; p.x_batch = (long)m.L * m.d;
        p.part = ws;
        LORY_TRY(k::launch_dense_stream_gu(st, p, m.B));
    }
    prof::Range r(st, prof::kGemmDown, 2.0 * m.tokens * m.D, 2.0 * (m.tokens * (double)m.d + (double)m.B * m.D));
    p.K = m.dff; p.N = m.d; p.ks = sp.down;
    p.W[0] = Wbar + (size_t)2 * m.B * m.D;
    p.gu = ws; p.gu_ks = sp.gu;
    p.part = parts;
    p.Y = Y; p.y_batch = (long)m.L * m.d;
    LORY_TRY(k::launch_dense_stream_down(st, p, m.B));
    if (sp.down > 1) LORY_TRY(k::launch_sum_store(st, parts, sp.down, m.B, (long)m.L * m.d, 1, Y, (long)m.L * m.d));
    return LORY_OK;
}

// Dense SwiGLU FFN of every sequence with its own materialised merged parameters
// (m.T == m.L: one parameter set per sequence, any number of rows).
int bf16_dense_ffn_fwd(const Dims &m, const void *Xv, const void *Wbarv, void *Yv, void *ws, size_t ws_bytes,
                       const DenseScratch &scratch, hipStream_t st)
{
    const bf *Wbar = (const bf *)Wbarv;
    const DensePlan pl = dense_plan(m, scratch);
    const int nt = pl.terms;
    bf *Act = (bf *)ws;
    float *parts = (float *)((char *)ws + pl.act);
    const long TD = (long)m.L * m.d;
    for (int r0 = 0; r0 < m.L; r0 += pl.rows) {
        const int rows = m.L - r0 < pl.rows ? m.L - r0 : pl.rows;
        const bf *X = (const bf *)Xv + (size_t)r0 * m.d;
        bf *Y = (bf *)Yv + (size_t)r0 * m.d;
        const long RD = (long)rows * m.d, RF = (long)rows * m.dff;   // a sequence's part of the block
        {
            const DenseSplit sp = pl.gate_up(m, rows);
            Params p = {};
            p.A[0] = X; p.a_batch[0] = TD; p.lda[0] = m.d;
            p.B[0] = Wbar; p.b_batch[0] = m.D; p.ldb[0] = m.dff;
            p.B[1] = Wbar + (size_t)m.B * m.D; p.b_batch[1] = m.D; p.ldb[1] = m.dff;
            p.M = rows; p.N = m.dff; p.K = m.d; p.batches = m.B;
            prof::Range r(st, prof::kGemmGU, gemm_flops(p, 2, 1), 2.0 * m.B * ((double)RD + 2.0 * m.D + (double)RF));
            if (const int ks = pl.stream_gu(m, rows)) {
                stream::Params q = {};
                q.M = rows; q.K = m.d; q.N = m.dff; q.ks = ks;
                q.W[0] = p.B[0]; q.W[1] = p.B[1]; q.w_batch = m.D;
                q.x = X; q.x_batch = TD;
                q.part = parts;
                LORY_TRY(k::launch_dense_stream_gu(st, q, m.B));
                LORY_TRY(k::launch_sum_act(st, parts, ks, m.B, RF, nt, Act));
            } else if (sp.ks) {
                p.ksplit = sp.ks;
                p.batches = m.B * sp.ks;
                const k::EpiPart<2> epi = {parts, sp.ks, m.B, rows, m.dff};
                LORY_TRY(k::launch_gu_split(st, p, epi, sp.rows));
                LORY_TRY(k::launch_sum_act(st, parts, sp.ks, m.B, RF, nt, Act));
            } else if (nt == 1) {
                EpiGU epi = {nullptr, nullptr, Act, rows, m.dff, 0};
                LORY_TRY(k::launch_gu(st, p, epi));
            } else {
                LORY_TRY(k::launch_gu2(st, p, k::EpiAct2{Act, rows, m.dff}));
            }
        }
        {
            // the two terms of an activation are blocks of rows of one matrix, or two sources
            const DenseSplit sp = pl.down(m, rows);
            Params p = pl.down_params(m, rows, ws, ws_bytes);
            p.A[0] = Act; p.A[1] = Act + RF; p.a_batch[0] = p.a_batch[1] = nt * RF; p.lda[0] = p.lda[1] = m.dff;
            p.B[0] = p.B[1] = Wbar + (size_t)2 * m.B * m.D; p.b_batch[0] = p.b_batch[1] = m.D; p.ldb[0] = p.ldb[1] = m.d;
            prof::Range r(st, prof::kGemmDown, gemm_flops(p, 1, 1), 2.0 * m.B * ((double)RF + (double)m.D + (double)RD));
            const EpiStore epi = {Y, TD, m.d};
            if (sp.ks) {
                p.M = nt * rows;
                p.ksplit = sp.ks;
                p.batches = m.B * sp.ks;
                const k::EpiPart<1> part = {parts, sp.ks, m.B, nt * rows, m.d};
                LORY_TRY(k::launch_down_split(st, p, part, sp.rows));
                LORY_TRY(k::launch_sum_store(st, parts, sp.ks, m.B, RD, nt, Y, TD));
            } else if (nt == 1) {
                LORY_TRY(k::launch_down(st, p, epi));
            } else {
                LORY_TRY(k::launch_down2(st, p, epi));
            }
        }
    }
    return LORY_OK;
}

int bf16_ffn_bwd(const Dims &m, const void *Xv, const float *w, const void *Wgv, const void *Wuv,
                 const void *Wdv, const void *dYv, const void *Gv, const void *Uv, const void *Wbarv,
                 void *dXv, void *dWg, void *dWu, void *dWd, int grad_dtype, int accumulate, float *dw,
                 void *ws, hipStream_t st)
{
    // saved merged parameters [Wg_bar | Wu_bar | Wd_bar]: no re-merge, the GEMMs read them in place
    const bf *Wbar = (const bf *)Wbarv;
    const bf *Wbar_g = Wbar, *Wbar_u = Wbar ? Wbar + (size_t)m.S * m.D : nullptr;
    const bf *Wbar_d = Wbar ? Wbar + (size_t)2 * m.S * m.D : nullptr;
    const Plan pl = make_plan(m);
    const bf *X = (const bf *)Xv, *Wg = (const bf *)Wgv, *Wu = (const bf *)Wuv, *Wd = (const bf *)Wdv;
    const bf *dY = (const bf *)dYv, *G = (const bf *)Gv, *U = (const bf *)Uv;
    bf *dX = (bf *)dXv;
    char *base = (char *)ws;
    bf *dG = (bf *)base, *dU = (bf *)(base + pl.act), *Act = (bf *)(base + 2 * pl.act);
    bf *Gr = (bf *)(base + 3 * pl.act), *Ur = (bf *)(base + 4 * pl.act);
    bf *slab = (bf *)(base + 5 * pl.act);
    float *partials = (float *)(base + 5 * pl.act + pl.slab_bwd);
    const long TD = (long)m.T * m.d, TF = (long)m.T * m.dff;
    const int grid = k::scatter_grid();
    const int grad_f32 = (grad_dtype == LORY_F32) ? 1 : 0;
    // token contractions with the merge inside the GEMM (no re-merged slabs); the per-segment weight
    // gradients still pass through the slab
    const Fused fused = Wbar || m.S > pl.Sc ? Fused{} : use_fused(m, true);
    // ... unless the expert-gradient kernel that keeps them on chip takes the shape (bf16 gradients
    // that overwrite; at most 16 experts)
    auto dw_params = [&](const bf *A, int lda, const bf *B, int ldb, const bf *W, void *dW, int M, int N) {
        fsg::Params q = {};
        q.A = (const uint16_t *)A; q.lda = lda;
        q.B = (const uint16_t *)B; q.ldb = ldb;
        q.W = (const uint16_t *)W; q.dW = (uint16_t *)dW;
        q.expert_stride = (long)m.D; q.ldw = N;
        q.w = w; q.E = m.E; q.T = m.T; q.S = m.S; q.M = M; q.N = N;
        return q;
    };
    const bool fused_dw = fused.da && use_fused_dw() && !grad_f32 && !accumulate &&
                          k::fused_dw_fits(dw_params(nullptr, m.dff, nullptr, m.d, nullptr, nullptr, m.dff, m.d)) &&
                          k::fused_dw_fits(dw_params(nullptr, m.d, nullptr, m.dff, nullptr, nullptr, m.d, m.dff));

    for (int s0 = 0; s0 < m.S; s0 += pl.Sc) {
        const int S = (m.S - s0 < pl.Sc) ? (m.S - s0) : pl.Sc;
        const float *wc = w + (size_t)s0 * m.E;
        const bf *Xc = X + (size_t)s0 * TD;
        const bf *dYc = dY + (size_t)s0 * TD;
        const int acc_dW = (accumulate || s0 > 0) ? 1 : 0;
        int partials_add = 0;

        const bf *Gc, *Uc;
        if (G && U) {
            Gc = G + (size_t)s0 * TF;
            Uc = U + (size_t)s0 * TF;
        } else if (fused.gate_up) {
            LORY_TRY(fused_gate_up(st, m, X, Wg, Wu, w, Gr, Ur, false));
            Gc = Gr;
            Uc = Ur;
        } else {
            // the backward slab region holds four slabs of nf_bwd columns, i.e. a gate and an
            // up slab of 2 * nf_bwd columns each
            const int step = 2 * pl.nf_bwd;
            for (int n0 = 0; n0 < m.dff; n0 += step) {
                const int nf = (m.dff - n0 < step) ? (m.dff - n0) : step;
                LORY_TRY(gate_up_block(st, m, S, Xc, wc, Wg, Wu, n0, nf, slab, Gr, Ur, nullptr));
            }
            Gc = Gr;
            Uc = Ur;
        }

        if (fused.da) {
            // dA = dY Wd_bar^T for all of d_ff at once (Wd[e] is [d_ff][d]: K contiguous), then the
            // SwiGLU backward pass: dG, dU, A
            LORY_TRY(fused_gemm(st, m, prof::kFusedDA,
                                fused_params(m, dY, nullptr, m.d, Wd, nullptr, m.d, w, m.dff, m.d, dG, m.dff), 1, false));
            prof::Range r2(st, prof::kSwigluBwd, 12.0 * m.tokens * m.dff, 2.0 * 6.0 * m.tokens * m.dff);
            LORY_TRY(k::launch_swiglu_bwd(st, Gc, Uc, dG, dU, Act, m.tokens, m.dff, 0, m.dff));
        }

        if (fused_dw) {
            // expert gradients and routing-weight inner products of the three matrices, the per-segment
            // weight gradients never leaving the CU; every workgroup-wave adds its inner products
            // to a slot of its own, matrix after matrix
            fsg::Params q[3] = {dw_params(Act, m.dff, dY, m.d, Wd, dWd, m.dff, m.d),
                                dw_params(X, m.d, dG, m.dff, Wg, dWg, m.d, m.dff),
                                dw_params(X, m.d, dU, m.dff, Wu, dWu, m.d, m.dff)};
            int slots = 0;
            for (int i = 0; i < 3; ++i) {
                q[i].partials = partials;
                q[i].partials_add = i > 0;
                slots = k::fused_dw_slots(q[i]);   // the same for the three matrices (M N is)
                const double n = (double)m.D;
                prof::Range r(st, prof::kFusedDW, 2.0 * m.tokens * n + 8.0 * m.S * 16 * n,
                              2.0 * (2.0 * m.E * n + (double)m.tokens * (m.d + m.dff)));
                LORY_TRY(k::launch_fused_dw(st, q[i]));
            }
            prof::Range r(st, prof::kDwReduce, (double)slots * m.S * m.E, 4.0 * slots * m.S * 16);
            LORY_TRY(k::launch_dw_reduce(st, partials, slots, m.S, 16, dw, m.S, m.E));
        }

        // ---- d_ff blocks: dA (+ SwiGLU backward), weight-gradient slabs, scatter
        for (int n0 = 0; !fused_dw && n0 < m.dff; n0 += pl.nf_bwd) {
            const int nf = (m.dff - n0 < pl.nf_bwd) ? (m.dff - n0) : pl.nf_bwd;
            const size_t blk = (size_t)S * m.d * nf;  // elements of one slab of this block
            bf *s_md = slab, *s_gd = slab + blk, *s_gg = slab + 2 * blk, *s_gu = slab + 3 * blk;
            const Rect rows_d = rect(m.D, m.d, n0, nf, 0, m.d);      // rows n0.. of Wd [d_ff, d]
            const Rect cols_f = rect(m.D, m.dff, 0, m.d, n0, nf);    // columns n0.. of Wg/Wu [d, d_ff]

            // dA = dY Wd_bar^T for these d_ff columns, then the SwiGLU backward pass: dG, dU, A
            int32_t *map = Wbar ? nullptr : map_place(S, s_gd, (char *)slab + pl.slab_bwd);   // the gradient slabs are written later
            if (!Wbar && !fused.da) LORY_TRY(merge(st, wc, S, m.E, Wd, rows_d, s_md, map));
            if (!fused.da) {
                Params p = da_gemm(m, pl, S, nf, slab);
                p.b_map = map;
                p.A[0] = dYc; p.a_batch[0] = TD; p.lda[0] = m.d;
                p.B[0] = Wbar ? Wbar_d + (size_t)n0 * m.d : s_md;
                p.b_batch[0] = Wbar ? m.D : (long)nf * m.d;
                p.ldb[0] = m.d;
                EpiStore epi = {dG + n0, TF, m.dff};  // dA parks in the dG buffer
                int rec;
                {
                    prof::Range r(st, prof::kGemmDA, gemm_flops(p, 1, 1),
                                  2.0 * ((double)S * TD + (double)S * nf * m.d + (double)S * m.T * nf));
                    rec = r.index();
                    LORY_TRY(k::launch_da(st, p, epi));
                }
                prof::shared_segments(st, rec, map, S, 2.0 * nf * m.d);
                prof::Range r2(st, prof::kSwigluBwd, 12.0 * S * m.T * nf, 2.0 * 6.0 * S * m.T * nf);
                LORY_TRY(k::launch_swiglu_bwd(st, Gc, Uc, dG, dU, Act, (long)S * m.T, m.dff, n0, nf));
            }
            // dWd_bar rows = A^T dY
            {
                Params p = {};
                p.A[0] = Act + n0; p.a_batch[0] = TF; p.lda[0] = m.dff;
                p.B[0] = dYc; p.b_batch[0] = TD; p.ldb[0] = m.d;
                p.M = nf; p.N = m.d; p.K = m.T; p.batches = S;
                EpiStore epi = {s_gd, (long)nf * m.d, m.d};
                prof::Range r(st, prof::kGemmDWD, gemm_flops(p, 1, 1),
                              2.0 * ((double)S * m.T * nf + (double)S * TD + (double)S * nf * m.d));
                LORY_TRY(k::launch_dwd(st, p, epi));
            }
            // dWg_bar, dWu_bar columns = X^T dG, X^T dU
            {
                Params p = {};
                p.A[0] = Xc; p.a_batch[0] = TD; p.lda[0] = m.d;
                p.B[0] = dG + n0; p.b_batch[0] = TF; p.ldb[0] = m.dff;
                p.B[1] = dU + n0; p.b_batch[1] = TF; p.ldb[1] = m.dff;
                p.M = m.d; p.N = nf; p.K = m.T; p.batches = S;
                EpiStore2 epi = {s_gg, s_gu, (long)m.d * nf, nf};
                prof::Range r(st, prof::kGemmDWGU, gemm_flops(p, 2, 1),
                              2.0 * ((double)S * TD + 2.0 * S * m.T * nf + 2.0 * S * m.d * nf));
                LORY_TRY(k::launch_dwgu(st, p, epi));
            }
            // E-way scatter and router-weight inner products
            const bf *stacks[3] = {Wd, Wg, Wu};
            void *grads[3] = {dWd, dWg, dWu};
            const bf *gsl[3] = {s_gd, s_gg, s_gu};
            const Rect rcs[3] = {rows_d, cols_f, cols_f};
            for (int i = 0; i < 3; ++i) {
                const int padd = partials_add;
                for (int e0 = 0; e0 < m.E; e0 += 32) {  // windows of 32 experts
                    ScatterParams sp;
                    sp.w = wc; sp.S = S; sp.E = m.E; sp.e0 = e0;
                    sp.gslab = gsl[i]; sp.seg_stride = (long)rcs[i].nr * rcs[i].nc;
                    sp.stack = stacks[i]; sp.dW = grads[i]; sp.rc = rcs[i];
                    sp.grad_f32 = grad_f32; sp.accumulate = acc_dW;
                    sp.partials = partials; sp.pcols = pl.pcol; sp.partials_add = padd;
                    const int win = (m.E - e0 < 32) ? (m.E - e0) : 32;
                    const double n = (double)rcs[i].nr * rcs[i].nc;
                    const double gsz = grad_f32 ? 4.0 : 2.0;
                    prof::Range r(st, prof::kScatter, 4.0 * S * win * n,
                                  2.0 * n * (S + win) + gsz * n * win * (acc_dW ? 2 : 1));
                    LORY_TRY(k::launch_scatter(st, sp, grid));
                }
                partials_add = 1;
            }
        }

        if (fused.dx) {
            // dX = dG Wg_bar^T + dU Wu_bar^T: two sources, Wg[e] / Wu[e] are [d][d_ff] (K contiguous)
            LORY_TRY(fused_gemm(st, m, prof::kFusedDX,
                                fused_params(m, dG, dU, m.dff, Wg, Wu, m.dff, w, m.d, m.dff, dX, m.d), 2, false));
        }
        // ---- dX = dG Wg_bar^T + dU Wu_bar^T, one block of d columns at a time
        for (int k0 = 0; !fused.dx && k0 < m.d; k0 += pl.kf_bwd) {
            const int kf = (m.d - k0 < pl.kf_bwd) ? (m.d - k0) : pl.kf_bwd;
            const size_t blk = (size_t)S * kf * m.dff;
            bf *s_g = slab, *s_u = slab + blk;
            const Rect rows = rect(m.D, m.dff, k0, kf, 0, m.dff);
            int32_t *map = Wbar ? nullptr : map_place(S, slab + 2 * blk, (char *)slab + pl.slab_bwd);
            if (!Wbar) {
                LORY_TRY(merge(st, wc, S, m.E, Wg, rows, s_g, map));
                LORY_TRY(merge(st, wc, S, m.E, Wu, rows, s_u, map));
            }
            Params p = dx_gemm(m, pl, S, kf, slab);
            p.b_map = map;
            p.A[0] = dG; p.a_batch[0] = TF; p.lda[0] = m.dff;
            p.A[1] = dU; p.a_batch[1] = TF; p.lda[1] = m.dff;
            p.B[0] = Wbar ? Wbar_g + (size_t)k0 * m.dff : s_g;
            p.B[1] = Wbar ? Wbar_u + (size_t)k0 * m.dff : s_u;
            p.b_batch[0] = p.b_batch[1] = Wbar ? m.D : (long)kf * m.dff;
            p.ldb[0] = p.ldb[1] = m.dff;
            EpiStore epi = {dX + (size_t)s0 * TD + k0, TD, m.d};
            int rec;
            {
                prof::Range r(st, prof::kGemmDX, gemm_flops(p, 1, 2),
                              2.0 * (2.0 * S * TF + 2.0 * S * kf * m.dff + (double)S * m.T * kf));
                rec = r.index();
                LORY_TRY(k::launch_dx(st, p, epi));
            }
            prof::shared_segments(st, rec, map, S, 4.0 * kf * m.dff);
        }

        if (!fused_dw) {
            int prow, pcol;
            k::scatter_partial_dims(S, m.E, &prow, &pcol);
            prof::Range r(st, prof::kDwReduce, (double)grid * S * m.E, 4.0 * grid * prow * pcol);
            LORY_TRY(k::launch_dw_reduce(st, partials, grid, prow, pcol, dw + (size_t)s0 * m.E, S, m.E));
        }
    }
    return LORY_OK;
}

}  // namespace lory
