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
// dR, a workgroup per 16 rows of R, a chain of loads and sums over the segments; beside it the HBM-bound
// read-modify-write of dX, a wavefront per segment, block of rows and 64 chunks of columns: no width leaves lanes idle but in the last
// columns, and all workgroups fit the chip at once (a workgroup per four rows of R and one per segment and block
// of rows did not beyond d = 2048).  us, two launches / a workgroup per segment and block of rows / now: 64 segments of 256 tokens,
// d = 2048, 32 experts 58 / 37 / 38; 16 of 1024, d = 2560, 8 experts 47 / 77 / 38; 32 sequences of two segments of
// 256, d = 1024, 16 experts 26 / 29 / 14; 448 segments of 64, d = 1536, 24 experts 104 / 82 / 52.
#include "lory_internal.h"

#include <hip/hip_bf16.h>

#include <type_traits>

namespace lory {

namespace {

constexpr int kDxThreads = 256;
constexpr int kWaves = kDxThreads / 64;
constexpr int kDrCols = 4;                 // rows of R of a wavefront, lane = expert
constexpr int kDrRows = kDrCols * kWaves;  // of a workgroup
constexpr int kDrChunk = 64;               // segments whose dz sit in LDS at a time
constexpr int kDxRows = 8;                 // rows of dX that a thread has in flight
// Wavefronts that share the work on dX, in blocks of at least 8 rows.  Each reads its columns of R once, and more of them share
// the memory less evenly: 115 layers took 1.02 of the time of the best of 768, 1024, 1280, 1536 and 2048 with 1536, 1.03 to
// 1.06 with the others.
constexpr long kDxWaves = 1536;

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

// <e, de> over the wavefront, lanes 32, 16, 8, 4, 2 and 1 apart added in this order, without LDS.  After the lanes 8 apart
// are added a row of 16 repeats itself, so that its rotation by 4 is the lane 4 apart, and so on.
__device__ __forceinline__ float wave_dot(float e, float de)
{
    const uint32_t p = __float_as_uint(e * de);
    const auto a = __builtin_amdgcn_permlane32_swap(p, p, false, false);   // {lower half twice, upper half twice}
    float x = fmaf(e, de, __uint_as_float((threadIdx.x & 32) ? a[0] : a[1]));
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(b[0]) + __uint_as_float(b[1]);
    auto ror = [](float v, auto n) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + n, 0xf, 0xf, true)); };
    x += ror(x, std::integral_constant<int, 8>());
    x += ror(x, std::integral_constant<int, 4>());
    x += ror(x, std::integral_constant<int, 2>());
    x += ror(x, std::integral_constant<int, 1>());
    return x;
}

// e (de - <e, de>) for lane = expert; every lane of the wavefront takes part, with zeros beyond the experts.
__device__ __forceinline__ float softmax_jacobian(float e, float de) { return e * (de - wave_dot(e, de)); }

// dz of segment s = b*N + j (j < N-1) for lane = expert.
__device__ __forceinline__ float softmax_jacobian_row(const float *__restrict__ w, const float *__restrict__ dw,
                                                      int s, int E, int lane)
{
    float e = 0.f, de = 0.f;
    if (lane < E) {
        e = w[(size_t)(s + 1) * E + lane];
        de = dw[(size_t)(s + 1) * E + lane];
    }
    return softmax_jacobian(e, de);
}

// Columns of dX for a wavefront: 16 bytes a lane, or one where rows are not whole 16-byte pieces.
template <typename T>
__host__ __device__ constexpr int wave_cols(int d) { return d % (16 / (int)sizeof(T)) == 0 ? 64 * (16 / (int)sizeof(T)) : 64; }

// Adds dhbar[s, :] / T to rows [rb * rows_per, ...) of segment s of dX, wave_cols columns from c0: the work of one wavefront.
template <typename T>
__device__ __forceinline__ void route_bwd_dx(const T *__restrict__ R, const float *__restrict__ w, const float *__restrict__ dw,
                                             T *__restrict__ dX, int Tseg, int d, int E, int rows_per, int s, int rb, int c0,
                                             float *dz)
{
    constexpr int VEC = 16 / (int)sizeof(T);  // elements per 16-byte access
    const int lane = threadIdx.x & 63;
    const int t0 = rb * rows_per;
    const int t1 = (t0 + rows_per < Tseg) ? (t0 + rows_per) : Tseg;
    const float invT = 1.0f / (float)Tseg;
    T *Xs = dX + (size_t)s * Tseg * d;
    const bool vec = d % VEC == 0;
    const int c = c0 + lane * VEC;

    // the first rows are on their way while the gradient of the mean is formed
    uint4 q[kDxRows];
    auto load_rows = [&](int t) {
#pragma unroll
        for (int u = 0; u < kDxRows; ++u)
            if (t + u < t1) q[u] = *reinterpret_cast<const uint4 *>(Xs + (size_t)(t + u) * d + c);
    };
    if (vec && c < d) load_rows(t0);
    dz[lane] = softmax_jacobian_row(w, dw, s, E, lane);   // read by this wavefront alone
    __builtin_amdgcn_wave_barrier();

    if (vec) {
        if (c < d) {
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
            for (int t = t0; t < t1; t += kDxRows) {
                uint4 v[kDxRows];
#pragma unroll
                for (int u = 0; u < kDxRows; ++u) v[u] = q[u];
                if (t + kDxRows < t1) load_rows(t + kDxRows);
#pragma unroll
                for (int u = 0; u < kDxRows; ++u)
                    if (t + u < t1) *reinterpret_cast<uint4 *>(Xs + (size_t)(t + u) * d + c) = update(v[u]);
            }
        }
    } else {
        const int k = c0 + lane;
        if (k < d) {
            const float dh = dot_row(R + (size_t)k * E, dz, E) * invT;
            for (int t = t0; t < t1; ++t) {
                T *p = Xs + (size_t)t * d + k;
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

// dR[c, e] (+)= sum over s in ascending order of hbar[s, c] * dz[s, e], c = kDrRows * block + kDrCols * wavefront + 0 .. 3, e = lane.
__device__ __forceinline__ void route_bwd_dr(const float *__restrict__ hbar, const float *__restrict__ w,
                                             const float *__restrict__ dw, float *__restrict__ dR, int S, int d, int E, int N,
                                             int accumulate, int block, float (*dz)[64])
{
    const int tid = threadIdx.x;
    const int e = tid & 63, wave = tid >> 6;
    const int c = block * kDrRows + wave * kDrCols;
    float acc[kDrCols];
#pragma unroll
    for (int k = 0; k < kDrCols; ++k) acc[k] = 0.f;
    // Lane sl holds the means of segment s0 + sl in this wavefront's columns; the rows of its sixteen segments (every fourth) are
    // in flight together (one that does not route reads row 0), those of the next chunk behind the products of this one.
    constexpr int kSegs = kDrChunk / kWaves;
    float h[kDrCols], we[kSegs], de[kSegs];
    auto routes = [&](int s) { return s < S && s % N != N - 1; };
    auto load = [&](int s0) {
#pragma unroll
        for (int g = 0; g < kSegs; g += 4) {
            if (s0 + g * kWaves >= S) break;
#pragma unroll
            for (int i = g; i < g + 4; ++i) {
                const int s = s0 + i * kWaves + wave;
                const size_t at = (size_t)(routes(s) ? s + 1 : 0) * E + (e < E ? e : 0);
                we[i] = w[at];
                de[i] = dw[at];
            }
        }
#pragma unroll
        for (int k = 0; k < kDrCols; ++k) {
            const bool ok = c + k < d && s0 + e < S;
            h[k] = hbar[ok ? (size_t)(s0 + e) * d + c + k : 0];
            if (!ok) h[k] = 0.f;
        }
    };
    load(0);
    for (int s0 = 0; s0 < S; s0 += kDrChunk) {
        float hs[kDrCols];
#pragma unroll
        for (int k = 0; k < kDrCols; ++k) hs[k] = h[k];
#pragma unroll
        for (int g = 0; g < kSegs; g += 4) {
            if (s0 + g * kWaves >= S) break;
#pragma unroll
            for (int i = g; i < g + 4; ++i) {
                const int s = s0 + i * kWaves + wave;
                const float v = softmax_jacobian(e < E ? we[i] : 0.f, e < E ? de[i] : 0.f);
                dz[i * kWaves + wave][e] = routes(s) ? v : 0.f;
            }
        }
        if (s0 + kDrChunk < S) load(s0 + kDrChunk);
        __syncthreads();
        for (int j0 = 0; j0 < kDrChunk && s0 + j0 < S; j0 += 8) {   // beyond S: zero times zero
            float z[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) z[j] = dz[j0 + j][e];
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
                for (int k = 0; k < kDrCols; ++k) acc[k] += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(hs[k]), j0 + j)) * z[j];
        }
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < kDrCols; ++k)
        if (c + k < d && e < E) {
            float *dst = dR + (size_t)(c + k) * E + e;
            *dst = accumulate ? (*dst + acc[k]) : acc[k];
        }
}

// Workgroups 0 .. dr_blocks - 1: dR (they start first: a chain of loads, few bytes); the others: dX, a wavefront for 64 chunks
// of columns in a block of rows of a segment that routes (all but the last of every sequence), columns first.
template <typename T>
__global__ __launch_bounds__(kDxThreads) void route_bwd_dx_kernel(const T *__restrict__ R, const float *__restrict__ w,
                                                               const float *__restrict__ hbar, const float *__restrict__ dw,
                                                               T *__restrict__ dX, float *__restrict__ dR, int S, int Tseg, int d,
                                                               int E, int N, int rows_per, int row_blocks, int accumulate, int dr_blocks)
{
    __shared__ float dz[kDrChunk][64];
    const int id = blockIdx.x;
    if (id < dr_blocks) {
        route_bwd_dr(hbar, w, dw, dR, S, d, E, N, accumulate, id, dz);
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), cols = wave_cols<T>(d);
    const int u = (id - dr_blocks) * kWaves + wave, col_blocks = (d + cols - 1) / cols;
    const int seg_row = u / col_blocks, seg = seg_row / row_blocks;
    if (seg >= S / N * (N - 1)) return;
    route_bwd_dx(R, w, dw, dX, Tseg, d, E, rows_per, seg / (N - 1) * N + seg % (N - 1), seg_row % row_blocks, u % col_blocks * cols, dz[wave]);
}

template <typename T>
int launch_route_bwd(const Dims &m, const void *R, const float *w, const float *hbar, const float *dw,
                     void *dX, float *dR, int accumulate, hipStream_t st)
{
    const int col_blocks = (m.d + wave_cols<T>(m.d) - 1) / wave_cols<T>(m.d), segs = m.S - m.B;
    long rb = segs > 0 ? (kDxWaves + (long)segs * col_blocks - 1) / ((long)segs * col_blocks) : 1;
    if (rb > m.T / 8) rb = m.T / 8;
    if (rb < 1) rb = 1;
    const int rows_per = (int)((m.T + rb - 1) / rb), row_blocks = (m.T + rows_per - 1) / rows_per;
    const int dr_blocks = (m.d + kDrRows - 1) / kDrRows;
    const long units = (long)segs * row_blocks * col_blocks;
    hipLaunchKernelGGL((route_bwd_dx_kernel<T>), dim3((unsigned)(dr_blocks + (units + kWaves - 1) / kWaves)), dim3(kDxThreads), 0, st, (const T *)R, w, hbar, dw,
                       (T *)dX, dR, m.S, m.T, m.d, m.E, m.N, rows_per, row_blocks, accumulate, dr_blocks);
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
