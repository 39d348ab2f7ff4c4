// Dense FFN of a few token rows per sequence (decode steps of prompt-only routing, paper Section 3.1):
// out[t][n] = sum_k x[t][k] W[k][n], W row-major, streamed from memory to the matrix instruction without passing
// through LDS.  gfx950, bf16 operands, fp32 accumulation.
//
// A workgroup owns 128 columns of one matrix of one sequence and a K slice; its wavefronts take the K steps of 32 in
// turn.  Lane (c, g) of a wavefront loads 8 consecutive columns of the 8 K rows 8 g .. 8 g + 7 of a step (256-byte
// pieces of a row per 16 lanes: a CU reads 43 GB/s from memory that way and 28 in 128-byte pieces) and transposes them
// in registers into the operand of v_mfma_f32_16x16x32_bf16, 8 K values of one column; the other operand is up to 16
// token rows.  The wavefronts' sums meet in LDS and are added in wavefront order, those of the K slices in slice order
// by whoever reads them (bit-reproducible): the down projection forms its slice of the activation from the gate/up
// sums while its first weights are in flight, so a call is two launches and, where the down projection is cut, a small
// third one that adds.
//
// Bound by the latency of memory for small matrices and by its read rate for large ones: a CU reads at most 25 .. 45 GB/s,
// so the K slices are cut until all 256 take part.  us per call, ring GEMM -> this, weights from memory: one sequence,
// one token, d = 1024, d_ff = 2816 (17 MB) 19.6 -> 15.1 launched from Python, 13.2 from C; 4 at d = 2048, d_ff = 5632
// (277 MB) 59.6 -> 51.4, 5.4 TB/s.  Unsplit, with the activation in the epilogue of gate/up, the
// same kernels took 21.2 for the first: too few CUs read.
//
// Gate/up alone also for 17 .. 63 rows, 2 .. 4 row blocks per wavefront against the same weights; their sums leave for the
// launch that forms the activation, and the down projection stays on the ring GEMM (the activation of that many rows in
// two terms does not fit in LDS beside its sums, and every column block would form it again).  The weights
// skip LDS, and a barrier per K step with it.  us per call, ring GEMM -> this: 2 x 40 rows at
// d = 2048, d_ff = 5632 52.1 -> 46.4, 2 x 50 at 1536, 4096 39.5 -> 36.9, 3 x 45 at 768, 2048 27.8 -> 25.5, 24 at 1024,
// 2816 21.7 -> 20.8, 18 .. 33 at 2048, 5632 unchanged; where its estimate is not lower the ring GEMM runs
// (dense_stream_gu_slices).  64 rows are slower (32.5 -> 34.4 at 2048, 5632), two workgroups sharing the rows of more are
// as well (2 x 100 63 -> 74: the weights pass through the CUs twice), and the accumulators of 96 rows spill.
#pragma once

#include "bf16_kernels.h"

namespace lory {
namespace stream {

using gemm::bf16x8;
using gemm::u32x4;
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kMaxRows = 16;
constexpr int kMaxGuRows = 63;   // of gate/up alone
constexpr int kCols = 128;   // columns of a workgroup

template <class F, int... D>
__device__ __forceinline__ void each_of(F &&f, std::integer_sequence<int, D...>)
{
    (f(std::integral_constant<int, D>()), ...);
}

// DOWN: x is formed from the gate/up sums and leaves as bf16 or, where the contraction is cut, as partial sums; else
// gate or up (blockIdx.z & 1), partial sums.  NW: wavefronts.  DEPTH: K steps of a wavefront in flight.
// MT: blocks of 16 rows.
template <bool DOWN, int NW, int DEPTH, int MT>
__global__ __launch_bounds__(NW * 64) void dense_stream_kernel(const Params p)
{
    static_assert(!DOWN || MT == 1, "the activation of a slice of many rows does not fit in LDS");
    constexpr int TERMS = DOWN ? 2 : 1, SETS = DOWN ? 1 : 2;
    constexpr int XF = DOWN ? TERMS : MT;   // row fragments of a step
    extern __shared__ __attribute__((aligned(16))) char smem[];
    uint16_t *act = reinterpret_cast<uint16_t *>(smem);   // DOWN: [2][M][slice]
    float *red = reinterpret_cast<float *>(smem);         // afterwards: [NW][M][kCols]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4;
    const int sl = blockIdx.y, b = blockIdx.z / SETS, set = blockIdx.z % SETS, batches = gridDim.z / SETS;
    const int n0 = blockIdx.x * kCols;
    const int nc = n0 + 8 * c < p.N ? n0 + 8 * c : p.N - 8;   // columns beyond the matrix are not stored
    auto row = [&](int t) { return 16 * t + c < p.M ? 16 * t + c : p.M - 1; };   // nor are rows beyond the block
    const int total = p.K / 32;
    const int s0 = (int)((long)total * sl / p.ks), steps = (int)((long)total * (sl + 1) / p.ks) - s0;
    const int len = steps * 32;

    // wave-uniform bases in scalar registers, 32-bit lane offsets
    const char *W = reinterpret_cast<const char *>(p.W[set] + (size_t)b * p.w_batch + (size_t)s0 * 32 * p.N);
    const uint32_t offW = 2u * ((uint32_t)(8 * g) * (uint32_t)p.N + (uint32_t)nc);
    const char *x = nullptr;
    if constexpr (!DOWN) x = reinterpret_cast<const char *>(p.x + (size_t)b * p.x_batch + s0 * 32);
    uint32_t offX[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t)
        offX[t] = DOWN ? (uint32_t)row(t) * (uint32_t)len + 8u * g : 2u * ((uint32_t)row(t) * (uint32_t)p.K + 8u * g);

    u32x4 wr[DEPTH][8];
    bf16x8 xr[DEPTH][XF];
    f32x4 acc[MT][8];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto load = [&](auto buf, int step) {
        const size_t k = (size_t)step * 32;
#pragma unroll
        for (int i = 0; i < 8; ++i)
            wr[buf][i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(W + (k + i) * p.N * 2 + offW));
        if constexpr (!DOWN) {
#pragma unroll
            for (int t = 0; t < MT; ++t) xr[buf][t] = *reinterpret_cast<const bf16x8 *>(x + 2 * k + offX[t]);
        }
    };
    auto multiply = [&](auto buf, int step) {
        if constexpr (DOWN) {
#pragma unroll
            for (int t = 0; t < TERMS; ++t)
                xr[buf][t] = *reinterpret_cast<const bf16x8 *>(act + (size_t)t * p.M * len + offX[0] + step * 32);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            union {
                uint32_t w[4];
                bf16x8 v;
            } o;   // column j of the lane's piece, K rows 8 g .. 8 g + 7
#pragma unroll
            for (int ip = 0; ip < 4; ++ip)
                o.w[ip] = __builtin_amdgcn_perm(wr[buf][2 * ip + 1][j >> 1], wr[buf][2 * ip][j >> 1],
                                                (j & 1) ? 0x07060302u : 0x05040100u);
#pragma unroll
            for (int t = 0; t < XF; ++t) {
                f32x4 &a = acc[DOWN ? 0 : t][j];
                a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xr[buf][t], o.v, a, 0, 0, 0);
            }
            if constexpr (MT > 1) __builtin_amdgcn_sched_barrier(0);   // one column at a time: keeps register use flat
        }
    };
    // the activation of the slice: gate/up sums added in slice order, two bf16 terms
    auto stage_act = [&]() {
        if constexpr (DOWN) {
            const int quads = p.M * len / 4;
            const size_t up = (size_t)p.M * p.K, pitch = (size_t)batches * 2 * up;
            for (int q = tid; q < quads; q += NW * 64) {
                const int t = q / (len / 4), k = (q - t * (len / 4)) * 4;
                const float *src = p.gu + ((size_t)b * 2 * p.M + t) * p.K + s0 * 32 + k;
                float4 sg = make_float4(0.f, 0.f, 0.f, 0.f), su = sg;
                // eight loads in flight: left to itself the compiler waits for each pair beside the weights' registers
                auto add = [&](auto count, int s) {
                    float4 a[count], u[count];
#pragma unroll
                    for (int i = 0; i < count; ++i) {
                        a[i] = *reinterpret_cast<const float4 *>(src + (s + i) * pitch);
                        u[i] = *reinterpret_cast<const float4 *>(src + (s + i) * pitch + up);
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int i = 0; i < count; ++i) {
                        sg.x += a[i].x; sg.y += a[i].y; sg.z += a[i].z; sg.w += a[i].w;
                        su.x += u[i].x; su.y += u[i].y; su.z += u[i].z; su.w += u[i].w;
                    }
                };
                int s = 0;
                for (; s + 4 <= p.gu_ks; s += 4) add(std::integral_constant<int, 4>(), s);
                if (p.gu_ks & 2) add(std::integral_constant<int, 2>(), s);
                if (p.gu_ks & 1) add(std::integral_constant<int, 1>(), p.gu_ks - 1);
                float h[4], l[4];
                k::act_terms(sg.x, su.x, h[0], l[0]);
                k::act_terms(sg.y, su.y, h[1], l[1]);
                k::act_terms(sg.z, su.z, h[2], l[2]);
                k::act_terms(sg.w, su.w, h[3], l[3]);
                uint16_t *dst = act + (size_t)t * len + k;
                *reinterpret_cast<gemm::u32x2 *>(dst) = k::pack4(h[0], h[1], h[2], h[3]);
                *reinterpret_cast<gemm::u32x2 *>(dst + (size_t)p.M * len) = k::pack4(l[0], l[1], l[2], l[3]);
            }
            __syncthreads();
        }
    };

    const int n = (steps - wave + NW - 1) / NW;   // this wavefront's steps: wave, wave + NW, ..
    auto nth = [&](int i) { return wave + i * NW; };
    auto each = [](auto f) { each_of(f, std::make_integer_sequence<int, DEPTH>()); };
    // The loop's loads are unconditional: behind a conditional load the compiler waits for everything in flight.
    if constexpr (MT > 1) {
        // One copy of the loop, or the accumulators move between registers at its ends.  Past the slice its last step is
        // loaded again, for nobody.
        auto at = [&](int i) { return nth(i) < steps ? nth(i) : steps - 1; };
        each([&](auto d) { load(d, at(d)); });
        int i = 0;
#pragma unroll 1
        for (; i + DEPTH <= n; i += DEPTH)
            each([&](auto d) {
                multiply(d, 0);
                load(d, at(i + DEPTH + d));
            });
        each([&](auto d) {
            if (i + d < n) multiply(d, 0);
        });
    } else {
        auto fill_full = [&]() { each([&](auto d) { load(d, nth(d)); }); };
        auto run_full = [&]() {
            int i = 0;
            for (; i + 2 * DEPTH <= n; i += DEPTH)
                each([&](auto d) {
                    multiply(d, nth(i + d));
                    load(d, nth(i + DEPTH + d));
                });
            const int left = n - i - DEPTH;   // steps that are not in flight yet, fewer than DEPTH
            each([&](auto d) {
                multiply(d, nth(i + d));
                if (d < left) load(d, nth(i + DEPTH + d));
            });
            each([&](auto d) {
                if (d < left) multiply(d, nth(i + DEPTH + d));
            });
        };
        auto fill_few = [&]() {
            each([&](auto d) {
                if (d < n) load(d, nth(d));
            });
        };
        auto run_few = [&]() {
            each([&](auto d) {
                if (d < n) multiply(d, nth(d));
            });
        };
        const bool full = n >= DEPTH;   // not the same for every wavefront of a workgroup
        if constexpr (DOWN) {
            if (full) fill_full();
            else fill_few();
            stage_act();   // holds a barrier: outside the arms, where every wavefront passes
            if (full) run_full();
            else run_few();
        } else if (full) {
            fill_full();
            run_full();
        } else {
            fill_few();
            run_few();
        }
    }

    // Lane (c, g) holds tokens 4 g .. 4 g + 3 of a row block, columns 8 c .. 8 c + 7.
    if constexpr (DOWN) __syncthreads();   // every wavefront has read its activation
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int tok = 16 * t + 4 * g + r;
            if (tok < p.M) {
#pragma unroll
                for (int j = 0; j < 8; j += 4)
                    *reinterpret_cast<float4 *>(red + (wave * p.M + tok) * kCols + 8 * c + j) =
                        make_float4(acc[t][j][r], acc[t][j + 1][r], acc[t][j + 2][r], acc[t][j + 3][r]);
            }
            if constexpr (MT > 1) __builtin_amdgcn_sched_barrier(0);
        }
    __syncthreads();
#pragma unroll 1
    for (int q = tid; q < p.M * (kCols / 4); q += NW * 64) {
        const int tok = q / (kCols / 4), col = q % (kCols / 4) * 4;
        if (n0 + col >= p.N) continue;
        float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float4 s = *reinterpret_cast<const float4 *>(red + (w * p.M + tok) * kCols + col);
            v[0] += s.x; v[1] += s.y; v[2] += s.z; v[3] += s.w;
        }
        if (!DOWN || p.ks > 1)
            *reinterpret_cast<float4 *>(p.part + ((((size_t)sl * batches + b) * SETS + set) * p.M + tok) * p.N + n0 + col) =
                make_float4(v[0], v[1], v[2], v[3]);
        else
            *reinterpret_cast<gemm::u32x2 *>(p.Y + (size_t)b * p.y_batch + (size_t)tok * p.N + n0 + col) =
                k::pack4(v[0], v[1], v[2], v[3]);
    }
}

template <bool DOWN, int NW>
constexpr size_t lds_bytes(int M, int steps, int ks)
{
    const size_t red = (size_t)NW * M * kCols * 4, act = DOWN ? (size_t)2 * M * ((steps + ks - 1) / ks) * 64 : 0;
    return red > act ? red : act;
}

template <bool DOWN, int NW, int DEPTH, int MT = 1>
inline hipError_t launch(hipStream_t st, const Params &p, int batches)
{
    const long z = (long)batches * (DOWN ? 1 : 2);
    if (p.M < 1 || p.M > 16 * MT || p.ks < 1 || p.ks > 65535 || p.ks > p.K / 32 || z > 65535 || p.K % 32 != 0 || p.N % 8 != 0 ||
        p.N < 8 || p.K >= (1 << 26) || p.N >= (1 << 26))
        return hipErrorInvalidValue;
    const size_t lds = lds_bytes<DOWN, NW>(p.M, p.K / 32, p.ks);
    if (lds > 160 * 1024) return hipErrorInvalidValue;
    auto kern = dense_stream_kernel<DOWN, NW, DEPTH, MT>;
    static bool configured = false;  // per instantiation
    if (!configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           160 * 1024);
        if (e != hipSuccess) return e;
        configured = true;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)((p.N + kCols - 1) / kCols), (unsigned)p.ks, (unsigned)z), dim3(NW * 64), lds, st, p);
    return hipGetLastError();
}

}  // namespace stream
}  // namespace lory
