// Instantiations of the merge / scatter / router-weight-gradient kernels.
#include "bf16_kernels.h"

namespace lory {
namespace k {

namespace {
// dw[s][e] = sum over slots of partials[slot][s][e].  One workgroup per segment row: thread
// (e, g) adds slots g, g+16, ... along four interleaved chains (fixed order), sixteen loads in flight, then the 16 group
// sums are added in order.
__global__ __launch_bounds__(1024) void dw_reduce_kernel(const float *__restrict__ partials, int slots,
                                                         int rows, int cols, float *__restrict__ dw,
                                                         int S, int E)
{
    __shared__ float red[16][64];
    const int s = blockIdx.x;
    const int e = threadIdx.x & 63, g = threadIdx.x >> 6;
    float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
    if (e < E) {
        const float *src = partials + (size_t)s * cols + e;
        const size_t pitch = (size_t)rows * cols;
        int k = g;
        for (; k + 240 < slots; k += 256) {
            float v[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = src[(size_t)(k + 16 * i) * pitch];
#pragma unroll
            for (int i = 0; i < 16; i += 4) {
                a0 += v[i];
                a1 += v[i + 1];
                a2 += v[i + 2];
                a3 += v[i + 3];
            }
        }
        for (; k + 48 < slots; k += 64) {
            a0 += src[(size_t)k * pitch];
            a1 += src[(size_t)(k + 16) * pitch];
            a2 += src[(size_t)(k + 32) * pitch];
            a3 += src[(size_t)(k + 48) * pitch];
        }
        for (; k < slots; k += 16) a0 += src[(size_t)k * pitch];
    }
    red[g][e] = (a0 + a1) + (a2 + a3);
    __syncthreads();
    if (g == 0 && e < E) {
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) sum += red[i][e];
        dw[(size_t)s * E + e] = sum;
    }
}

constexpr int kMsGrid = 1024;  // workgroups; 4 wavefronts each stride over the 256-element units

int units_of(const ms::Rect &rc) { return ((rc.nr * rc.nc / 8) + 31) / 32; }
}  // namespace

int scatter_grid() { return kMsGrid; }

namespace {
int kbm_of(int S)
{
    const int KB = (S + 15) / 16;
    int kbm = 1;
    while (kbm < KB) kbm *= 2;
    return kbm;
}
}  // namespace

void scatter_partial_dims(int S, int E, int *rows, int *cols)
{
    *rows = kbm_of(S) * 16;
    *cols = ((E + 31) / 32) * 32;
}

// Rounds of workgroups of a merge of `elems` parameters (one workgroup fits a CU).  Each round pays for a start
// (routing-weight operands, first loads: 3 us), several even out what the CUs get done.  What is uneven are the stores: beside the
// E streams that it reads, a wavefront writes S, and up to about ten more than a quarter of its reads a single round is the fastest
// at every size.  Beyond, the gain grows with the bytes of those stores, twice as fast into merged parameters
// that are kept as into the slab that the GEMM behind the merge reads (`transient`), part of which the memory-side cache holds.
// The lines are fitted to 803 prompt merges (S = 1 .. 64, 4 .. 32 experts, 768 x 768 .. 2560 x 6144) and 393 forward passes
// (S = 4 .. 128) in one, two and four rounds: 0.2 % slower than the fastest on average, 6 and 3 % at most (moved by 15 %
// either way the average stays); one round everywhere 1.1 and 0.7 %, 18 and 7 %, four 11 and 7 %, 41 and 24 %.
// us in one / two / four rounds: 3 prompts, 16 experts, 2048 x 5632 281 / 282 / 295; 64 sequences, 12 experts, 1024 x 2816
// 291 / 275 / 250.
int merge_rounds(int E, int S, long elems, bool transient)
{
    const double mb = 2e-6 * elems * (S - 10 - 0.25 * E) * (transient ? 0.5 : 1.0);
    return mb < 75 ? 1 : mb < 190 ? 2 : 4;
}

hipError_t launch_merge(hipStream_t st, const ms::MergeParams &p)
{
    const int KS = (p.E + 15) / 16;
    const int MB = (p.S + 31) / 32;
    const size_t lds = (size_t)MB * KS * 2 * 64 * 16;
    if (lds > 64 * 1024) return hipErrorInvalidValue;
    const int most = merge_rounds(p.E, p.S, (long)p.rc.nr * p.rc.nc, p.seg_map != nullptr) * gemm2::cu_count();
    int grid = (units_of(p.rc) + 3) / 4;
    if (grid > most) grid = most;
#define LORY_MERGE(K)                                                                              \
    if (p.seg_map)                                                                                 \
        hipLaunchKernelGGL((ms::merge_kernel<K, true>), dim3(grid), dim3(256), lds, st, p);        \
    else                                                                                           \
        hipLaunchKernelGGL((ms::merge_kernel<K, false>), dim3(grid), dim3(256), lds, st, p)
    switch (KS) {
    case 1: LORY_MERGE(1); break;
    case 2: LORY_MERGE(2); break;
    case 3: LORY_MERGE(3); break;
    case 4: LORY_MERGE(4); break;
    default: return hipErrorInvalidValue;
    }
#undef LORY_MERGE
    return hipGetLastError();
}

// One unit a wavefront takes a merge as long as a unit's registers hold all segments: 8, and 16 with up to 8 experts (whose
// unit is twice as large).  us of the three merges of a layer, merge_kernel and merge_few_kernel: 3 prompts, 16 experts of
// 2048 x 5632 273 and 216; 8 and 14 of 2048 x 6144 322 and 273; 16 and 6 of 1536 x 4096 175 and 135; 16 and 6 of 2048 x 5632
// 285 and 254.  Forward passes, with the GEMMs that read the slab: 8 segments, 48 experts of 1024 x 2816 272 and 209;
// 15 and 8 of 1536 x 2816 252 and 228; 16 and 7 of 2048 x 5632 636 and 619.  38 layers on average 0.83 of the time, the worst
// 0.96 (backward 0.92 and 0.98).
bool merge_is_few(int S, int E)
{
    return S <= (E <= 8 ? ms::kFewSegments : 8);
}

hipError_t launch_merge_few(hipStream_t st, const ms::MergeFewParams &p, int matrices)
{
    if (p.S < 1 || !merge_is_few(p.S, p.E) || p.E < 1 || p.E > 64 || matrices < 1 || matrices > 3) return hipErrorInvalidValue;
    const int chunks = 4 * ms::few_unit_chunks(p.E);   // of a workgroup
    const dim3 grid((unsigned)((p.rc.nr * p.rc.nc / 8 + chunks - 1) / chunks), (unsigned)matrices);
#define LORY_FEW(K, N)                                                                               \
    if (p.seg_map)                                                                                   \
        hipLaunchKernelGGL((ms::merge_few_kernel<K, N, true>), grid, dim3(256), 0, st, p);           \
    else                                                                                             \
        hipLaunchKernelGGL((ms::merge_few_kernel<K, N, false>), grid, dim3(256), 0, st, p)
    switch (p.E <= 8 ? 0 : (p.E + 15) / 16) {
    case 0:
        if (p.S > 8) {
            LORY_FEW(0, 8);
        } else {
            LORY_FEW(0, 4);
        }
        break;
    case 1: LORY_FEW(1, 4); break;
    case 2: LORY_FEW(2, 4); break;
    case 3: LORY_FEW(3, 4); break;
    default: LORY_FEW(4, 4); break;
    }
#undef LORY_FEW
    return hipGetLastError();
}

hipError_t launch_scatter(hipStream_t st, const ms::ScatterParams &p, int grid)
{
    const int KB = (p.S + 15) / 16;
    if (KB > 16 || p.e0 % 32 != 0 || p.e0 >= p.E) return hipErrorInvalidValue;
    const int win = (p.E - p.e0 < 32) ? (p.E - p.e0) : 32;
    const int eb16 = (win + 15) / 16;
    const size_t lds_main = (size_t)KB * 2 * 64 * 16 + 4 * 16 * ms::kDotPitch;
#define LORY_SCATTER(K, B)                                                                            \
    do {                                                                                              \
        const size_t lds_red = (size_t)4 * K * B * 1024;                                              \
        const size_t lds_work = lds_main + (ms::scatter_parks_experts<K, B>() ? 4 * B * 4096 : 0);    \
        const size_t lds = lds_work > lds_red ? lds_work : lds_red;                                   \
        auto kern = ms::scatter_kernel<K, B>;                                                         \
        if (lds > 48 * 1024) {                                                                        \
            static bool configured = false;                                                           \
            if (!configured) {                                                                        \
                hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),              \
                                                   hipFuncAttributeMaxDynamicSharedMemorySize,        \
                                                   160 * 1024);                                       \
                if (e != hipSuccess) return e;                                                        \
                configured = true;                                                                    \
            }                                                                                         \
        }                                                                                             \
        hipLaunchKernelGGL(kern, dim3(grid), dim3(256), lds, st, p);                                  \
    } while (0)
#define LORY_SCATTER_K(B)                          \
    switch (kbm_of(p.S)) {                         \
    case 1: LORY_SCATTER(1, B); break;             \
    case 2: LORY_SCATTER(2, B); break;             \
    case 4: LORY_SCATTER(4, B); break;             \
    case 8: LORY_SCATTER(8, B); break;             \
    default: LORY_SCATTER(16, B); break;           \
    }
    if (eb16 == 1) {
        LORY_SCATTER_K(1)
    } else {
        LORY_SCATTER_K(2)
    }
#undef LORY_SCATTER_K
#undef LORY_SCATTER
    return hipGetLastError();
}

hipError_t launch_dw_reduce(hipStream_t st, const float *partials, int slots, int rows, int cols,
                            float *dw, int S, int E)
{
    hipLaunchKernelGGL(dw_reduce_kernel, dim3(S), dim3(1024), 0, st, partials, slots, rows, cols, dw, S,
                       E);
    return hipGetLastError();
}

}  // namespace k
}  // namespace lory
