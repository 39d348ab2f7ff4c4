// Launch wrappers of the bf16 kernels; each group of instantiations lives in a
// translation unit of its own so that they compile in parallel.
#pragma once

#include "lory_internal.h"
#include "gemm_bf16.h"
#include "gemm2_bf16.h"
#include "merge_scatter_bf16.h"
#include "fused_bf16.h"
#include "fused_bwd_bf16.h"

namespace lory {
namespace stream {

// One projection of the streaming dense FFN (dense_stream_bf16.h).
struct Params {
    int M, K, N;           // rows per sequence; K a multiple of 32, N of 8
    int ks;                // K slices of the contraction
    const uint16_t *W[2];  // [batches][K][N]: gate and up, or down
    long w_batch;
    const uint16_t *x;     // gate/up: token rows x + b * x_batch + m * K
    long x_batch;
    const float *gu;       // down: gate/up sums [gu_ks][batches][2][M][K]
    int gu_ks;
    float *part;           // sums [ks][batches][matrices][M][N] (gate/up; down where ks > 1)
    uint16_t *Y;           // down where ks == 1: Y + b * y_batch + m * N
    long y_batch;
};

}  // namespace stream

namespace k {

using gemm::bf16_bits_to_float;
using gemm::float_to_bf16_bits;

using gemm::u32x2;

__device__ __forceinline__ u32x2 pack4(float a, float b, float c, float d)
{
    u32x2 r;
    r.x = gemm::cvt_pk_bf16(a, b);
    r.y = gemm::cvt_pk_bf16(c, d);
    return r;
}

// Gate/up projections of one column block of d_ff: planes A = silu(G) * U, G, U.
// SAVE: write G and U; ACT: write A.  (Compile-time so that the epilogue has no data-dependent
// control flow.)
template <bool SAVE, bool ACT>
struct EpiGUT {
    static constexpr int NOUT = 3;
    static constexpr bool SPLIT = false, TAIL = false;
    uint16_t *G, *U, *Act;  // [tokens, d_ff]
    int T, dff, n_off;
    __device__ __forceinline__ bool enabled(int o) const { return o == 0 ? ACT : SAVE; }
    __device__ __forceinline__ u32x2 pack(int o, const float (&v)[2][4]) const
    {
        if (o == 1) return pack4(v[0][0], v[0][1], v[0][2], v[0][3]);
        if (o == 2) return pack4(v[1][0], v[1][1], v[1][2], v[1][3]);
        float a[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] = v[0][e] * __builtin_amdgcn_rcpf(1.0f + __expf(-v[0][e])) * v[1][e];
        return pack4(a[0], a[1], a[2], a[3]);
    }
    __device__ __forceinline__ long row_bytes() const { return 2L * dff; }
    __device__ __forceinline__ uint16_t *ptr(int o, int s, int m, int n) const
    {
        uint16_t *base = (o == 0) ? Act : (o == 1) ? G : U;
        return base + ((size_t)s * T + m) * dff + n_off + n;
    }
};

// Run-time description of the same epilogue (G and U may both be NULL, Act may be NULL).
struct EpiGU {
    uint16_t *G, *U, *Act;
    int T, dff, n_off;
};

// An activation of fp32 precision as two bf16 terms, hi + lo (relative error up to 2^-18): the matrix instruction
// multiplies both with the same weights.  hi is the rounded value, or the truncated one where rounding would
// overflow; infinities and NaN go into hi alone.  Error of the dense FFN against 64 bits, activation in fp32 on the
// vector ALUs / these two terms / rounded to bf16, 1e-3: 2 x 100 tokens at d = 2048, d_ff = 5632 1.659371 / 1.659373 /
// 2.344863, one token at d = 1024, d_ff = 2816 1.611728 / 1.611738 / 2.262393 (the rounding of the output is 1.66).
__device__ __forceinline__ void act_terms(float g, float u, float &hi, float &lo)
{
    const float a = g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u;   // 32 bits: 3e-7 for |g| < 4
    const uint32_t bits = __float_as_uint(a);
    uint32_t h = gemm::cvt_pk_bf16(a, 0.f) << 16;
    const bool finite = (bits & 0x7f800000u) != 0x7f800000u;
    if (finite && (h & 0x7f800000u) == 0x7f800000u) h = bits & 0xffff0000u;
    hi = __uint_as_float(h);
    lo = finite ? a - hi : 0.f;
}

// Gate/up projections, activation as two terms: Act[batch][hi rows | lo rows][d_ff].
struct EpiAct2 {
    static constexpr int NOUT = 2;
    static constexpr bool SPLIT = false, TAIL = false;
    uint16_t *Act;
    int T, dff;
    __device__ __forceinline__ bool enabled(int) const { return true; }
    __device__ __forceinline__ u32x2 pack(int o, const float (&v)[2][4]) const
    {
        float t[2][4];
#pragma unroll
        for (int e = 0; e < 4; ++e) act_terms(v[0][e], v[1][e], t[0][e], t[1][e]);
        return o == 0 ? pack4(t[0][0], t[0][1], t[0][2], t[0][3]) : pack4(t[1][0], t[1][1], t[1][2], t[1][3]);
    }
    __device__ __forceinline__ long row_bytes() const { return 2L * dff; }
    __device__ __forceinline__ uint16_t *ptr(int o, int s, int m, int n) const
    {
        return Act + ((size_t)(2 * s + o) * T + m) * dff + n;
    }
};

// C[batch][m][n] = bf16(v)
struct EpiStore {
    static constexpr int NOUT = 1;
    static constexpr bool SPLIT = false, TAIL = true;
    uint16_t *C;
    long c_batch;
    int ldc;
    __device__ __forceinline__ bool enabled(int) const { return true; }
    __device__ __forceinline__ u32x2 pack(int, const float (&v)[1][4]) const
    {
        return pack4(v[0][0], v[0][1], v[0][2], v[0][3]);
    }
    __device__ __forceinline__ long row_bytes() const { return 2L * ldc; }
    __device__ __forceinline__ uint16_t *ptr(int, int b, int m, int n) const
    {
        return C + (size_t)b * c_batch + (size_t)m * ldc + n;
    }
};

// The same for two operand sets: C0 from the first, C1 from the second.
struct EpiStore2 {
    static constexpr int NOUT = 2;
    static constexpr bool SPLIT = false, TAIL = false;
    uint16_t *C0, *C1;
    long c_batch;
    int ldc;
    __device__ __forceinline__ bool enabled(int) const { return true; }
    __device__ __forceinline__ u32x2 pack(int o, const float (&v)[2][4]) const
    {
        return o == 0 ? pack4(v[0][0], v[0][1], v[0][2], v[0][3]) : pack4(v[1][0], v[1][1], v[1][2], v[1][3]);
    }
    __device__ __forceinline__ long row_bytes() const { return 2L * ldc; }
    __device__ __forceinline__ uint16_t *ptr(int o, int b, int m, int n) const
    {
        return (o == 0 ? C0 : C1) + (size_t)b * c_batch + (size_t)m * ldc + n;
    }
};

// fp32 partial sums of one K slice: part[slice][batch][set][m][n]
template <int NSET>
struct EpiPart {
    static constexpr int NOUT = 1;
    static constexpr bool SPLIT = true, TAIL = false;
    float *P;
    int ksplit, batches, M, N;   // batches: items before the split
    __device__ __forceinline__ bool enabled(int) const { return false; }
    __device__ __forceinline__ long row_bytes() const { return 0; }
    __device__ __forceinline__ uint16_t *ptr(int, int, int, int) const { return nullptr; }
    __device__ __forceinline__ u32x2 pack(int, const float (&)[NSET][4]) const { return u32x2{0, 0}; }
    __device__ __forceinline__ float *part(int set, int bs, int m, int n) const
    {
        const int sl = bs % ksplit, b = bs / ksplit;
        return P + ((((size_t)sl * batches + b) * NSET + set) * M + m) * N + n;
    }
};

// Every wrapper returns a hipError_t.  Any M (a multiple of 8 where A is stored K-slow), N a multiple of 8,
// K a multiple of 32 and at least 64.
int merge_rounds(int E, int S, long elems, bool transient);   // rounds of workgroups that launch_merge starts
hipError_t launch_merge(hipStream_t st, const ms::MergeParams &p);
bool merge_is_few(int S, int E);          // whether launch_merge_few takes the merge of S segments
hipError_t launch_merge_few(hipStream_t st, const ms::MergeFewParams &p, int matrices);
hipError_t launch_scatter(hipStream_t st, const ms::ScatterParams &p, int grid);
hipError_t launch_dw_reduce(hipStream_t st, const float *partials, int slots, int rows, int cols,
                            float *dw, int S, int E);
int scatter_grid();                       // workgroups the scatter kernel is launched with
void scatter_partial_dims(int S, int E, int *rows, int *cols);

// merge inside the GEMM (fused_bf16.h): C = sum over nsrc sources of A_q * Wbar_q(segment of the row)
bool fused_fits(const fmg::Params &p);
hipError_t launch_fused(hipStream_t st, const fmg::Params &p, int nsrc, bool w_nc);
// two products of A[0] with N-contiguous stacks: C = A[0] Wbar_0, C2 = A[0] Wbar_1
hipError_t launch_fused_pair(hipStream_t st, const fmg::Params &p);
// the same with fp32 C and C2, on the eight-wave kernel only
hipError_t launch_fused_pair_f32(hipStream_t st, const fmg::Params &p);

// expert gradients and routing-weight inner products with the per-segment weight gradients kept on
// chip (fused_bwd_bf16.h); the partial-sum buffer holds fused_dw_slots(p) x S x 16 floats
bool fused_dw_fits(const fsg::Params &p);
int fused_dw_slots(const fsg::Params &p);
hipError_t launch_fused_dw(hipStream_t st, const fsg::Params &p);

hipError_t launch_gu(hipStream_t st, const gemm::Params &p, const EpiGU &e);     // X * [Wg_bar | Wu_bar]
hipError_t launch_gu2(hipStream_t st, const gemm::Params &p, const EpiAct2 &e);   // the same, activation as two terms
hipError_t launch_down(hipStream_t st, const gemm::Params &p, const EpiStore &e);  // A * Wd_bar
hipError_t launch_down2(hipStream_t st, const gemm::Params &p, const EpiStore &e);  // A_hi * Wd_bar + A_lo * Wd_bar
// The same two projections with the contraction split into p.ksplit slices (p.batches already counts them);
// rows: tile height, 64 or 128.
hipError_t launch_gu_split(hipStream_t st, const gemm::Params &p, const EpiPart<2> &e, int rows);
hipError_t launch_down_split(hipStream_t st, const gemm::Params &p, const EpiPart<1> &e, int rows);
// Sums of the K slices in slice order.  part [ksplit][batches][2][mn] -> Act [batches][terms][mn], silu(G) * U
// rounded (terms = 1) or as two terms; part [ksplit][batches][terms][mn] -> Y, mn elements every y_batch.
hipError_t launch_sum_act(hipStream_t st, const float *part, int ksplit, long batches, long mn, int terms, uint16_t *Act);
hipError_t launch_sum_store(hipStream_t st, const float *part, int ksplit, long batches, long mn, int terms, uint16_t *Y,
                            long y_batch);
// Dense FFN of at most 16 rows per sequence (dense_stream_bf16.h): K slices of its two projections, both 0 where it
// does not take the call (more rows, or partial sums that `floats` do not hold).
DenseStream dense_stream_plan(int B, int M, int d, int dff, size_t floats);
// Its gate/up projections alone, for 17 .. 63 rows: K slices, 0 where it does not take them or the ring GEMM, in its
// estimated time, is not slower.
int dense_stream_gu_slices(int B, int M, int d, int dff, size_t floats, double ring_us);
hipError_t launch_dense_stream_gu(hipStream_t st, const stream::Params &p, int B);
hipError_t launch_dense_stream_down(hipStream_t st, const stream::Params &p, int B);

hipError_t launch_da(hipStream_t st, const gemm::Params &p, const EpiStore &e);  // dY * Wd_bar^T
hipError_t launch_swiglu_fwd_f32(hipStream_t st, const float *G, const float *U, uint16_t *Act, long elements);
hipError_t launch_swiglu_fwd(hipStream_t st, const uint16_t *G, const uint16_t *U, uint16_t *Act, long rows,
                             int dff, int n0, int nf);
hipError_t launch_swiglu_bwd(hipStream_t st, const uint16_t *G, const uint16_t *U, uint16_t *dG_dA,
                             uint16_t *dU, uint16_t *Act, long rows, int dff, int n0, int nf);
hipError_t launch_dx(hipStream_t st, const gemm::Params &p, const EpiStore &e);  // dG Wg_bar^T + dU Wu_bar^T
hipError_t launch_dwgu(hipStream_t st, const gemm::Params &p, const EpiStore2 &e);  // X^T [dG | dU]
hipError_t launch_dwd(hipStream_t st, const gemm::Params &p, const EpiStore &e);  // A^T dY

}  // namespace k
}  // namespace lory
