// SwiGLU forward and backward as streaming passes (HBM-bound).  Backward: from dA (left in the dG buffer by the
// dA = dY Wd_bar^T GEMM) and the saved G, U it produces, for one block of d_ff columns,
//   dG = dA * U * sig(G) * (1 + G (1 - sig(G))),  dU = dA * G * sig(G),  A = G sig(G) U
// (derivative of the LLaMA-style SwiGLU that the paper's experts use, Section 4.1).
#include "bf16_kernels.h"

namespace lory {
namespace k {

namespace {

__device__ __forceinline__ void unpack8(const uint4 &q, float (&f)[8])
{
    const uint32_t r[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[2 * i] = __uint_as_float(r[i] << 16);
        f[2 * i + 1] = __uint_as_float(r[i] & 0xffff0000u);
    }
}

__device__ __forceinline__ uint4 pack8(const float (&f)[8])
{
    uint4 q;
    q.x = gemm::cvt_pk_bf16(f[0], f[1]);
    q.y = gemm::cvt_pk_bf16(f[2], f[3]);
    q.z = gemm::cvt_pk_bf16(f[4], f[5]);
    q.w = gemm::cvt_pk_bf16(f[6], f[7]);
    return q;
}

// rows x (nf / 8) chunks of 8 columns; all arrays have row pitch dff and start at column n0.
__global__ __launch_bounds__(256) void swiglu_bwd_kernel(const uint16_t *__restrict__ G,
                                                         const uint16_t *__restrict__ U,
                                                         uint16_t *__restrict__ dG_dA,
                                                         uint16_t *__restrict__ dU,
                                                         uint16_t *__restrict__ Act, long rows, int dff,
                                                         int n0, int nf)
{
    const int cpr = nf >> 3;
    const long total = rows * cpr;
    for (long idx = (long)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
         idx += (long)gridDim.x * blockDim.x) {
        const long row = idx / cpr;
        const int c = (int)(idx - row * cpr) << 3;
        const size_t off = (size_t)row * dff + n0 + c;
        float g[8], u[8], da[8], og[8], ou[8], oa[8];
        unpack8(*reinterpret_cast<const uint4 *>(G + off), g);
        unpack8(*reinterpret_cast<const uint4 *>(U + off), u);
        unpack8(*reinterpret_cast<const uint4 *>(dG_dA + off), da);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float sg = __builtin_amdgcn_rcpf(1.0f + __expf(-g[i]));
            oa[i] = g[i] * sg * u[i];
            og[i] = da[i] * u[i] * sg * (1.0f + g[i] * (1.0f - sg));
            ou[i] = da[i] * g[i] * sg;
        }
        *reinterpret_cast<uint4 *>(dG_dA + off) = pack8(og);
        *reinterpret_cast<uint4 *>(dU + off) = pack8(ou);
        *reinterpret_cast<uint4 *>(Act + off) = pack8(oa);
    }
}

// A = G * sigmoid(G) * U for one block of d_ff columns (SwiGLU forward, Section 4.1).
__global__ __launch_bounds__(256) void swiglu_fwd_kernel(const uint16_t *__restrict__ G,
                                                         const uint16_t *__restrict__ U,
                                                         uint16_t *__restrict__ Act, long rows, int dff,
                                                         int n0, int nf)
{
    const int cpr = nf >> 3;
    const long total = rows * cpr;
    for (long idx = (long)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
         idx += (long)gridDim.x * blockDim.x) {
        const long row = idx / cpr;
        const int c = (int)(idx - row * cpr) << 3;
        const size_t off = (size_t)row * dff + n0 + c;
        float g[8], u[8], oa[8];
        unpack8(*reinterpret_cast<const uint4 *>(G + off), g);
        unpack8(*reinterpret_cast<const uint4 *>(U + off), u);
#pragma unroll
        for (int i = 0; i < 8; ++i) oa[i] = g[i] * __builtin_amdgcn_rcpf(1.0f + __expf(-g[i])) * u[i];
        *reinterpret_cast<uint4 *>(Act + off) = pack8(oa);
    }
}

// The same from fp32 G and U, contiguous: nothing is rounded before the activation itself.  HBM-bound, 10 bytes an element.
__global__ __launch_bounds__(256) void swiglu_fwd_f32_kernel(const float4 *__restrict__ G, const float4 *__restrict__ U,
                                                             uint4 *__restrict__ Act, long total)
{
    for (long idx = (long)blockIdx.x * blockDim.x + threadIdx.x; idx < total; idx += (long)gridDim.x * blockDim.x) {
        const float4 g0 = G[2 * idx], g1 = G[2 * idx + 1], u0 = U[2 * idx], u1 = U[2 * idx + 1];
        const float g[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
        const float u[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
        float oa[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) oa[i] = g[i] * __builtin_amdgcn_rcpf(1.0f + __expf(-g[i])) * u[i];
        Act[idx] = pack8(oa);
    }
}

// Sums of fp32 partial products over the K slices of a split contraction, in slice order, of NP planes `plane`
// apart; four consecutive elements per thread.  HBM-bound (the parts of a small call sit in the memory-side cache).
template <int NP>
__device__ __forceinline__ void sum_parts(const float *p, size_t plane, int ksplit, size_t pitch, float4 (&a)[NP])
{
#pragma unroll
    for (int j = 0; j < NP; ++j) a[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    int s = 0;
    for (; s + 4 <= ksplit; s += 4) {  // loads overlap, adds stay in order
        float4 v[4][NP];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < NP; ++j) v[i][j] = *reinterpret_cast<const float4 *>(p + (size_t)(s + i) * pitch + j * plane);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                a[j].x += v[i][j].x; a[j].y += v[i][j].y; a[j].z += v[i][j].z; a[j].w += v[i][j].w;
            }
    }
    for (; s < ksplit; ++s)
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const float4 v = *reinterpret_cast<const float4 *>(p + (size_t)s * pitch + j * plane);
            a[j].x += v.x; a[j].y += v.y; a[j].z += v.z; a[j].w += v.w;
        }
}

// part [ksplit][batches][2][mn] -> Act [batches][TERMS][mn]
template <int TERMS>
__global__ __launch_bounds__(256) void sum_act_kernel(const float *__restrict__ part, int ksplit, long batches, long mn,
                                                      uint16_t *__restrict__ Act)
{
    const long i = ((long)blockIdx.x * 256 + threadIdx.x) * 4;
    if (i >= batches * mn) return;
    const long b = i / mn, e = i - b * mn;
    const float *p = part + (size_t)b * 2 * mn + e;
    const size_t pitch = (size_t)batches * 2 * mn;
    float4 gu[2];
    sum_parts<2>(p, mn, ksplit, pitch, gu);
    const float4 g = gu[0], u = gu[1];
    if constexpr (TERMS == 1) {
        auto act = [](float x, float y) { return x * __builtin_amdgcn_rcpf(1.0f + __expf(-x)) * y; };
        *reinterpret_cast<u32x2 *>(Act + i) = pack4(act(g.x, u.x), act(g.y, u.y), act(g.z, u.z), act(g.w, u.w));
    } else {
        float h[4], l[4];
        act_terms(g.x, u.x, h[0], l[0]);
        act_terms(g.y, u.y, h[1], l[1]);
        act_terms(g.z, u.z, h[2], l[2]);
        act_terms(g.w, u.w, h[3], l[3]);
        uint16_t *dst = Act + (size_t)b * 2 * mn + e;
        *reinterpret_cast<u32x2 *>(dst) = pack4(h[0], h[1], h[2], h[3]);
        *reinterpret_cast<u32x2 *>(dst + mn) = pack4(l[0], l[1], l[2], l[3]);
    }
}

// part [ksplit][batches][TERMS][mn] -> Y, mn elements every y_batch
template <int TERMS>
__global__ __launch_bounds__(256) void sum_store_kernel(const float *__restrict__ part, int ksplit, long batches, long mn,
                                                        uint16_t *__restrict__ Y, long y_batch)
{
    const long i = ((long)blockIdx.x * 256 + threadIdx.x) * 4;
    if (i >= batches * mn) return;
    const long b = i / mn, e = i - b * mn;
    const float *p = part + (size_t)b * TERMS * mn + e;
    float4 y[TERMS];
    sum_parts<TERMS>(p, mn, ksplit, (size_t)batches * TERMS * mn, y);
#pragma unroll
    for (int j = 1; j < TERMS; ++j) {
        y[0].x += y[j].x; y[0].y += y[j].y; y[0].z += y[j].z; y[0].w += y[j].w;
    }
    *reinterpret_cast<u32x2 *>(Y + (size_t)b * y_batch + e) = pack4(y[0].x, y[0].y, y[0].z, y[0].w);
}

}  // namespace

hipError_t launch_sum_act(hipStream_t st, const float *part, int ksplit, long batches, long mn, int terms, uint16_t *Act)
{
    const dim3 grid((unsigned)((batches * mn / 4 + 255) / 256));
    if (terms == 1)
        hipLaunchKernelGGL(sum_act_kernel<1>, grid, dim3(256), 0, st, part, ksplit, batches, mn, Act);
    else
        hipLaunchKernelGGL(sum_act_kernel<2>, grid, dim3(256), 0, st, part, ksplit, batches, mn, Act);
    return hipGetLastError();
}

hipError_t launch_sum_store(hipStream_t st, const float *part, int ksplit, long batches, long mn, int terms, uint16_t *Y,
                            long y_batch)
{
    const dim3 grid((unsigned)((batches * mn / 4 + 255) / 256));
    if (terms == 1)
        hipLaunchKernelGGL(sum_store_kernel<1>, grid, dim3(256), 0, st, part, ksplit, batches, mn, Y, y_batch);
    else
        hipLaunchKernelGGL(sum_store_kernel<2>, grid, dim3(256), 0, st, part, ksplit, batches, mn, Y, y_batch);
    return hipGetLastError();
}

hipError_t launch_swiglu_fwd(hipStream_t st, const uint16_t *G, const uint16_t *U, uint16_t *Act, long rows,
                             int dff, int n0, int nf)
{
    const long total = rows * (nf / 8);
    long blocks = (total + 255) / 256;
    if (blocks > 256 * 16) blocks = 256 * 16;
    hipLaunchKernelGGL(swiglu_fwd_kernel, dim3((unsigned)blocks), dim3(256), 0, st, G, U, Act, rows, dff, n0, nf);
    return hipGetLastError();
}

hipError_t launch_swiglu_fwd_f32(hipStream_t st, const float *G, const float *U, uint16_t *Act, long elements)
{
    const long total = elements / 8;
    long blocks = (total + 255) / 256;
    if (blocks > 256 * 16) blocks = 256 * 16;
    hipLaunchKernelGGL(swiglu_fwd_f32_kernel, dim3((unsigned)blocks), dim3(256), 0, st,
                       reinterpret_cast<const float4 *>(G), reinterpret_cast<const float4 *>(U),
                       reinterpret_cast<uint4 *>(Act), total);
    return hipGetLastError();
}

hipError_t launch_swiglu_bwd(hipStream_t st, const uint16_t *G, const uint16_t *U, uint16_t *dG_dA,
                             uint16_t *dU, uint16_t *Act, long rows, int dff, int n0, int nf)
{
    const long total = rows * (nf / 8);
    long blocks = (total + 255) / 256;
    if (blocks > 256 * 16) blocks = 256 * 16;
    hipLaunchKernelGGL(swiglu_bwd_kernel, dim3((unsigned)blocks), dim3(256), 0, st, G, U, dG_dA, dU, Act,
                       rows, dff, n0, nf);
    return hipGetLastError();
}

}  // namespace k
}  // namespace lory
