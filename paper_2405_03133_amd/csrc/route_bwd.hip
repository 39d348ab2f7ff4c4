// Backward of the causal segment routing on gfx950 (chain rule through paper
// Section 3.1 / Eq. 2; stop gradient on the first segment as in Algorithm 1).
//
// Forward: e[b,j] = softmax(hbar[b,j] R), w[b,0] = sg(e[b,0]), w[b,k] = e[b,k-1].
// Given dw (gradient with respect to the routing weights w of every segment):
//   de[b,j]   = dw[b,j+1] for j < N-1, 0 for the last segment of a sequence
//               (dw[b,0] is dropped: that use of e[b,0] sits behind the stop gradient)
//   dz[b,j]   = e[b,j] (.) (de[b,j] - <e[b,j], de[b,j]>)          softmax Jacobian
//   dR        = sum over segments of hbar[b,j]^T dz[b,j]
//   dhbar     = dz R^T,  dX[b, jT+t, :] += dhbar[b,j,:] / T        mean broadcast
// e[b,j] is read back from the forward's output as w[b,j+1]; the last segment's
// e is never needed because its dz is zero.
//
// One launch of two kinds of workgroups, both with fixed summation orders (bit-reproducible): the tiny [d, S] x [S, E] product
// dR, a workgroup per four rows of R, and beside it the HBM-bound read-modify-write of dX, a workgroup per segment and
// block of rows.  64 segments of 256 tokens at d = 2048, 32 experts: 38 us (two launches, the rows loaded after the
// gradient of the mean: 42 + 12).
#include "lory_internal.h"

#include <hip/hip_bf16.h>

namespace lory {

namespace {

constexpr int kDxThreads = 256;
constexpr int kDrRows = kDxThreads / 64;   // rows of R of a workgroup: one for each wavefront, lane = expert
constexpr int kDrChunk = 64;               // segments whose dz sit in LDS at a time
constexpr int kDxRows = 8;                 // rows of dX that a thread has in flight

__device__ __forceinline__ float bf16_to_f32(uint16_t v) { return __uint_as_float((uint32_t)v << 16); }

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f)
{
    const uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);  // NaN stays NaN
    return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

__device__ __forceinline__ float load_elem(const float *p) { return *p; }
__device__ __forceinline__ float load_elem(const __hip_bfloat16 *p)
{
    return bf16_to_f32(*reinterpret_cast<const uint16_t *>(p));
}

// <dz, one row of R>: 16-byte loads when the row length allows it.
__device__ __forceinline__ float dot_row(const float *__restrict__ row, const float *dz, int E)
{
    float acc = 0.f;
    if (E % 4 == 0) {
        for (int e = 0; e < E; e += 4) {
            const float4 v = *reinterpret_cast<const float4 *>(row + e);
            acc += dz[e] * v.x + dz[e + 1] * v.y + dz[e + 2] * v.z + dz[e + 3] * v.w;
        }
    } else {
        for (int e = 0; e < E; ++e) acc += dz[e] * row[e];
    }
    return acc;
}
__device__ __forceinline__ float dot_row(const __hip_bfloat16 *__restrict__ row, const float *dz, int E)
{
    float acc = 0.f;
    if (E % 8 == 0) {
        for (int e = 0; e < E; e += 8) {
            const uint4 q = *reinterpret_cast<const uint4 *>(row + e);
            const uint32_t r[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int i = 0; i < 4; ++i)
                acc += dz[e + 2 * i] * __uint_as_float(r[i] << 16) +
                       dz[e + 2 * i + 1] * __uint_as_float(r[i] & 0xffff0000u);
        }
    } else {
        for (int e = 0; e < E; ++e) acc += dz[e] * load_elem(row + e);
    }
    return acc;
}

// dz of segment s = b*N + j (j < N-1) for lane = expert; every lane of the wavefront takes part.
__device__ __forceinline__ float softmax_jacobian_row(const float *__restrict__ w, const float *__restrict__ dw,
                                                      int s, int E, int lane)
{
    float e = 0.f, de = 0.f;
    if (lane < E) {
        e = w[(size_t)(s + 1) * E + lane];
        de = dw[(size_t)(s + 1) * E + lane];
    }
    float inner = e * de;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) inner += __shfl_xor(inner, off, 64);
    return e * (de - inner);
}

// Adds dhbar[s, :] / T to rows [rb * rows_per, ...) of segment s of dX.
template <typename T>
__device__ __forceinline__ void route_bwd_dx(const T *__restrict__ R, const float *__restrict__ w, const float *__restrict__ dw,
                                             T *__restrict__ dX, int Tseg, int d, int E, int N, int rows_per, int s, int rb,
                                             float *dz)
{
    constexpr int VEC = 16 / (int)sizeof(T);  // elements per 16-byte access
    if (s % N == N - 1) return;  // nothing routes on the last segment of a sequence
    const int tid = threadIdx.x;
    const int t0 = rb * rows_per;
    const int t1 = (t0 + rows_per < Tseg) ? (t0 + rows_per) : Tseg;
    const float invT = 1.0f / (float)Tseg;
    T *Xs = dX + (size_t)s * Tseg * d;
    const bool vec = d % VEC == 0;

    // the first rows are on their way while the gradient of the mean is formed
    uint4 q[kDxRows];
    auto load_rows = [&](int c, int t) {
#pragma unroll
        for (int u = 0; u < kDxRows; ++u)
            if (t + u < t1) q[u] = *reinterpret_cast<const uint4 *>(Xs + (size_t)(t + u) * d + c);
    };
    if (vec && tid * VEC < d) load_rows(tid * VEC, t0);
    if (tid < 64) dz[tid] = softmax_jacobian_row(w, dw, s, E, tid);
    __syncthreads();

    if (vec) {
        for (int c = tid * VEC; c < d; c += kDxThreads * VEC) {
            float dh[VEC];
#pragma unroll
            for (int i = 0; i < VEC; ++i) dh[i] = dot_row(R + (size_t)(c + i) * E, dz, E) * invT;
            auto update = [&](uint4 q) {
                if constexpr (sizeof(T) == 4) {
                    q.x = __float_as_uint(__uint_as_float(q.x) + dh[0]);
                    q.y = __float_as_uint(__uint_as_float(q.y) + dh[1]);
                    q.z = __float_as_uint(__uint_as_float(q.z) + dh[2]);
                    q.w = __float_as_uint(__uint_as_float(q.w) + dh[3]);
                    return q;
                } else {
                    uint32_t r[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float lo = __uint_as_float(r[i] << 16) + dh[2 * i];
                        const float hi = __uint_as_float(r[i] & 0xffff0000u) + dh[2 * i + 1];
                        r[i] = (uint32_t)f32_to_bf16_rne(lo) | ((uint32_t)f32_to_bf16_rne(hi) << 16);
                    }
                    return make_uint4(r[0], r[1], r[2], r[3]);
                }
            };
            if (c != tid * VEC) load_rows(c, t0);
            for (int t = t0; t < t1; t += kDxRows) {
                uint4 v[kDxRows];
#pragma unroll
                for (int u = 0; u < kDxRows; ++u) v[u] = q[u];
                if (t + kDxRows < t1) load_rows(c, t + kDxRows);
#pragma unroll
                for (int u = 0; u < kDxRows; ++u)
                    if (t + u < t1) *reinterpret_cast<uint4 *>(Xs + (size_t)(t + u) * d + c) = update(v[u]);
            }
        }
    } else {
        for (int c = tid; c < d; c += kDxThreads) {
            const float dh = dot_row(R + (size_t)c * E, dz, E) * invT;
            for (int t = t0; t < t1; ++t) {
                T *p = Xs + (size_t)t * d + c;
                if constexpr (sizeof(T) == 4) {
                    *p += dh;
                } else {
                    uint16_t *q = reinterpret_cast<uint16_t *>(p);
                    *q = f32_to_bf16_rne(bf16_to_f32(*q) + dh);
                }
            }
        }
    }
}

// dR[c, e] (+)= sum over s in ascending order of hbar[s, c] * dz[s, e], c = kDrRows * block + wavefront, e = lane.
__device__ __forceinline__ void route_bwd_dr(const float *__restrict__ hbar, const float *__restrict__ w,
                                             const float *__restrict__ dw, float *__restrict__ dR, int S, int d, int E, int N,
                                             int accumulate, int block, float (*dz)[64])
{
    const int tid = threadIdx.x;
    const int e = tid & 63, wave = tid >> 6;
    const int c = block * kDrRows + wave;
    float acc = 0.f;
    for (int s0 = 0; s0 < S; s0 += kDrChunk) {
        // lane sl holds the mean of segment s0 + sl in this wavefront's column
        const float h = (c < d && s0 + e < S) ? hbar[(size_t)(s0 + e) * d + c] : 0.f;
#pragma unroll
        for (int i = 0; i < kDrChunk / kDrRows; ++i) {
            const int sl = wave * (kDrChunk / kDrRows) + i;
            const int s = s0 + sl;
            float v = 0.f;
            if (s < S && (s % N) != N - 1) v = softmax_jacobian_row(w, dw, s, E, e);
            dz[sl][e] = v;
        }
        __syncthreads();
        const int n = (S - s0 < kDrChunk) ? (S - s0) : kDrChunk;
        for (int sl = 0; sl < n; ++sl) acc += __shfl(h, sl, 64) * dz[sl][e];
        __syncthreads();
    }
    if (c < d && e < E) {
        float *dst = dR + (size_t)c * E + e;
        *dst = accumulate ? (*dst + acc) : acc;
    }
}

// Workgroups 0 .. dr_blocks - 1: dR (they start first: a chain of loads, few bytes); the others: dX, segment by segment for
// each block of rows.
template <typename T>
__global__ __launch_bounds__(kDxThreads) void route_bwd_dx_kernel(const T *__restrict__ R, const float *__restrict__ w,
                                                               const float *__restrict__ hbar, const float *__restrict__ dw,
                                                               T *__restrict__ dX, float *__restrict__ dR, int S, int Tseg, int d,
                                                               int E, int N, int rows_per, int accumulate, int dr_blocks)
{
    __shared__ float dz[kDrChunk][64];
    const int id = blockIdx.x;
    if (id < dr_blocks)
        route_bwd_dr(hbar, w, dw, dR, S, d, E, N, accumulate, id, dz);
    else
        route_bwd_dx(R, w, dw, dX, Tseg, d, E, N, rows_per, (id - dr_blocks) % S, (id - dr_blocks) / S, dz[0]);
}

template <typename T>
int launch_route_bwd(const Dims &m, const void *R, const float *w, const float *hbar, const float *dw,
                     void *dX, float *dR, int accumulate, hipStream_t st)
{
    // Row blocks of at least 8 rows.  Each reads all of R in 16-byte pieces of its rows, so a large router takes one workgroup
    // for each CU, a small one four (us of the launch with 1024, 512 and 256 workgroups: 64 segments of 256 tokens, 32
    // experts, d = 2048 50, 48, 38; the fp32 configuration, d = 64 and 4 experts, 5.2, 6.2, 5.6).
    const int blocks = (long)m.d * m.E >= 8192 ? 256 : 1024;
    int rb = (blocks + m.S - 1) / m.S;
    if (rb > m.T / 8) rb = m.T / 8;
    if (rb < 1) rb = 1;
    const int rows_per = (m.T + rb - 1) / rb;
    rb = (m.T + rows_per - 1) / rows_per;
    const int dr_blocks = (m.d + kDrRows - 1) / kDrRows;
    hipLaunchKernelGGL((route_bwd_dx_kernel<T>), dim3(dr_blocks + m.S * rb), dim3(kDxThreads), 0, st, (const T *)R, w, hbar, dw,
                       (T *)dX, dR, m.S, m.T, m.d, m.E, m.N, rows_per, accumulate, dr_blocks);
    return launch_status();
}

}  // namespace

int route_bwd_launch(const Dims &m, const void *R, const float *w, const float *hbar, const float *dw,
                     void *dX, float *dR, int accumulate, hipStream_t st)
{
    if (m.dtype == LORY_F32) return launch_route_bwd<float>(m, R, w, hbar, dw, dX, dR, accumulate, st);
    return launch_route_bwd<__hip_bfloat16>(m, R, w, hbar, dw, dX, dR, accumulate, st);
}

}  // namespace lory
