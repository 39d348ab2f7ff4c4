// Types and helpers shared by the bf16 matrix-core kernels (gfx950): vector types, the problem statement
// of a batched GEMM, conversions between fp32 and bf16.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace lory {
namespace gemm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

struct Params {
    const uint16_t *A[2];  // per source
    long a_batch[2];       // elements between consecutive batch items
    int lda[2];            // elements between consecutive rows of the stored matrix
    const uint16_t *B[2];  // per operand set (NSET == 2) or per source (NSRC == 2)
    long b_batch[2];
    int ldb[2];
    const int32_t *b_map;  // batch item whose B operand an item reads, or NULL: its own
    int M, N, K;           // per batch item; K per source
    int batches;           // split contraction: ksplit entries per batch item
    int ksplit;            // K slices per batch item (split epilogues only)
    float *tail;           // scratch for the partial sums of a last round of tiles that is cut over K, or NULL
    size_t tail_floats;
    int pieces;            // set by the launch: K slices of a tile of that round (0: none is cut)
};

__device__ __forceinline__ float bf16_bits_to_float(uint16_t b)
{
    return __uint_as_float(((uint32_t)b) << 16);
}

// Round to nearest even; inputs here are finite.
__device__ __forceinline__ uint16_t float_to_bf16_bits(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// Two floats -> two bf16 (round to nearest even) packed into 32 bits, low half first: a single
// v_cvt_pk_bf16_f32 on gfx950.
__device__ __forceinline__ uint32_t cvt_pk_bf16(float lo, float hi)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const f32x2 v = {lo, hi};
    union {
        bf16x2 b;
        uint32_t u;
    } r;
    r.b = __builtin_convertvector(v, bf16x2);
    return r.u;
}

}  // namespace gemm
}  // namespace lory
