// Persistent batched bf16 MFMA GEMM for gfx950: 256-column tiles fed by an LDS ring that is filled
// with direct global->LDS loads (global_load_lds_dwordx4), so that two to three K steps of operands are
// in flight while one is being multiplied.  Every dense contraction of the merged FFN and of its backward
// (paper Section 3.1: o_x = FFN(h_x; theta_bar) for all tokens of a segment; Appendix B counts them as
// 6*L*d*d' FLOPs) is an instance of
//
//     C_b[M,N] = sum over sources q of  A_{q,b}[M,K] * B_{q,b}[K,N]
//
// with one batch item per segment and fp32 accumulation on v_mfma_f32_32x32x16_bf16.
//
// Operand layouts, chosen per instance by template flags:
//   A: "KC" = stored [M][K] (K contiguous)   or "MC" = stored [K][M]
//   B: "KC" = stored [N][K] (K contiguous)   or "NC" = stored [K][N]
//
// Any M and N (N a multiple of 8, M too for an MC operand): the loads of an edge tile are clamped to the
// last row or 16-byte chunk of the matrix and its stores are masked.  K % 32 == 0, at least two K steps.
//
// Per K step (BK = 32) a stage holds A (64 bytes per row of the tile) and B (16 KB).  A direct load
// writes the 64 lanes' 16-byte chunks to 1 KB of consecutive LDS, so the swizzles below are applied on
// the global side: each lane fetches the chunk that belongs at its LDS position.
//   K-contiguous operand: rows of 32 bf16 = 4 chunks; chunk c of row r lives in
//     slot c ^ f(r), f(r) = ((r>>1 ^ r>>3) & 1) | ((r>>2 & 1) << 1).
//   operand stored with K as the slow index (read with ds_read_b64_tr_b16, i.e. transposed by the LDS
//     read): 32 K rows of W bf16, dense; the 64-byte granule g of row k lives at granule g ^ ftr(k).
#pragma once

#include "gemm_bf16.h"

namespace lory {
namespace gemm2 {

using gemm::bf16x8;
using gemm::f32x16;
using gemm::Params;
using gemm::s16x4;
using gemm::u32x2;
using gemm::u32x4;

constexpr int BK = 32;
constexpr int kMaxCutK = 1 << 24;   // a contraction cut over K finds its slices in 32-bit arithmetic

// A tile shape: WMV x WNV wavefronts, each with MI x NB blocks of 32 x 32 outputs (NB counted through the
// operand sets), and the stages of its ring.  One workgroup per CU.
template <int WMV_, int WNV_, int MI_, int NB_, int STAGES>
struct Tile {
    static constexpr int WMV = WMV_, WNV = WNV_, MI = MI_, NB = NB_;
    static constexpr int NW = WMV * WNV;
    static constexpr int threads = NW * 64;
    static constexpr int BM = WMV * MI * 32;        // rows
    static constexpr int BN = WNV * NB * 32;        // columns over all operand sets
    static constexpr int stages = STAGES;
    static constexpr int waves_per_simd = NW / 4;
    static constexpr int a_bytes = BM * 64;
    static constexpr int b_bytes = BN * 64;
    static constexpr int stage = a_bytes + b_bytes;
    static constexpr int ring = stages * stage;
    static constexpr int JG = 2;                    // 32-column blocks staged at a time in the epilogue
    static constexpr int stage_out = 32 * JG * 64;  // bytes per wave
    static constexpr int total = ring + NW * stage_out;
    static_assert(a_bytes % (NW * 1024) == 0 && b_bytes % (NW * 1024) == 0, "every wave fetches whole kilobytes");
    static_assert(total <= 160 * 1024, "LDS of a CU");
};

__device__ __forceinline__ int fkc(int row)
{
    return (((row >> 1) ^ (row >> 3)) & 1) | (((row >> 2) & 1) << 1);
}

// XOR of the 64-byte granule index in row k of a K-slow tile W columns wide: the four rows that half a
// wave of a transposing read touches then lie in different banks.
template <int W>
__device__ __forceinline__ int ftr(int k)
{
    static_assert(W == 64 || W % 128 == 0, "a K-slow tile is 64 or a multiple of 128 columns wide");
    return W == 64 ? ((k >> 1) & 1) : (k & 3);
}

__device__ __forceinline__ bf16x8 frag_kc(const char *lds, int row0, int kk, int lane)
{
    const int row = row0 + (lane & 31);
    const int c = kk * 2 + (lane >> 5);
    return *reinterpret_cast<const bf16x8 *>(lds + row * 64 + ((c ^ fkc(row)) << 4));
}

__device__ __forceinline__ bf16x8 frag_tr(const char *p, int hi_off)
{
    typedef __attribute__((address_space(3))) s16x4 *lds_ptr;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p + hi_off));
    union {
        s16x4 h[2];
        bf16x8 v;
    } u;
    u.h[0] = lo;
    u.h[1] = hi;
    return u.v;
}

// One direct global->LDS load: every lane supplies its own global address, the 64 lanes'
// 16-byte chunks land at lds_addr + 16 * lane (lds_addr is wave-uniform and travels in M0).
// Issued as inline assembly so that the compiler's wait-count bookkeeping does not see an LDS
// writer: completion is tracked by hand with vmcnt below (VMEM operations of a wave retire in
// order), which is what lets three K steps stay in flight across barriers.
__device__ __forceinline__ void dma16(const uint16_t *g, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                 :
                 : "s"(lds_addr), "v"(g)
                 : "memory", "m0");
}

// The same with a wave-uniform base in scalar registers and a 32-bit byte offset per lane: a K step
// advances the base with one scalar addition and the lanes' offsets stay as they are.
__device__ __forceinline__ void dma16s(const char *base, uint32_t off, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(lds_addr), "v"(off), "s"(base)
                 : "memory", "m0");
}

// A wave-uniform pointer, for the compiler to see as one.
__device__ __forceinline__ const char *uniform(const char *p)
{
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (const char *)(((uint64_t)hi << 32) | lo);
}

template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Workgroup barrier without the release/acquire fence of __syncthreads() (which would wait for
// every outstanding load): LDS reads of this wave have returned (lgkmcnt) before it arrives.
__device__ __forceinline__ void ring_barrier()
{
    // s_waitcnt lgkmcnt(0) as a builtin (simm16 0xC07F: vmcnt and expcnt left at their maxima) so
    // that the compiler's own LDS bookkeeping knows the reads have returned.
    __builtin_amdgcn_s_waitcnt(0xC07F);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Persistent kernel: the grid is one workgroup per CU; every workgroup walks its own list of tiles, and the K
// steps of consecutive tiles form one stream through the ring, so the first operands of the next tile are already
// in flight while the current tile is multiplied and written out.
//
// TAIL: the tiles that do not fill a round of workgroups are cut into p.pieces K slices, one for each
// workgroup after its whole tiles; their fp32 sums go to p.tail and tail_kernel adds them and runs the epilogue.
template <int NSET, int NSRC, bool A_MC, bool B_NC, bool TAIL, class TL, class Epi>
__global__ __launch_bounds__(TL::threads, TL::waves_per_simd) void gemm2_kernel(const Params p, const Epi epi)
{
    static_assert(NSET == 1 || NSRC == 1, "either two operand sets or two sources");
    static_assert(!TAIL || !Epi::SPLIT, "all tiles or those of the last round are cut");
    constexpr int MI = TL::MI, NB = TL::NB;
    constexpr int BM = TL::BM;
    constexpr int BNS = TL::BN / NSET;    // columns per operand set
    constexpr int NI = NB / NSET;         // 32-column blocks per wave and set
    constexpr int WM = MI * 32;           // rows per wave
    constexpr int WN = NI * 32;           // columns per wave and set
    constexpr int S = TL::stages;
    constexpr int BSET_BYTES = TL::b_bytes / NSET;
    constexpr int LA = TL::a_bytes / (TL::NW * 1024), LB = TL::b_bytes / (TL::NW * 1024);  // direct loads of a wave per K step

    extern __shared__ __attribute__((aligned(16))) char smem[];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = (wave / TL::WNV) * WM;
    const int wn0 = (wave % TL::WNV) * WN;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;

    // Workgroups are dealt round-robin to the 8 XCDs (each with its own L2).  Every XCD gets a
    // contiguous range of tiles, shared cyclically by its workgroups, so that the tiles of one
    // segment, which share the A operand, meet in the same L2.
    const int tiles_n = (p.N + BNS - 1) / BNS;
    const int tiles_m = (p.M + BM - 1) / BM;
    const int ntiles = p.batches * tiles_m * tiles_n;
    const int whole = TAIL ? ntiles / (int)gridDim.x * (int)gridDim.x : ntiles;   // tiles that are not cut
    const int per_xcd = (whole + 7) >> 3;
    const int wg_per_xcd = gridDim.x >> 3;
    const int xcd = blockIdx.x & 7, qx = blockIdx.x >> 3;
    int xcd_tiles = whole - xcd * per_xcd;  // tiles in this XCD's range
    if (xcd_tiles > per_xcd) xcd_tiles = per_xcd;
    const int my_whole = (xcd_tiles > qx) ? (xcd_tiles - qx + wg_per_xcd - 1) / wg_per_xcd : 0;
    const int piece = xcd * wg_per_xcd + qx;   // this workgroup's K slice of the cut tiles, slices of a tile adjacent
    const int my_tiles = my_whole + ((TAIL && piece < (ntiles - whole) * p.pieces) ? 1 : 0);
    if (my_tiles == 0) return;

    const int ktiles = p.K / BK;
    // K steps of a tile, at least two.  Epi::SPLIT: a batch item's contraction is cut into ksplit slices that
    // count as batch items of their own (index b * ksplit + slice) and leave as fp32 partial sums.
    static_assert(!Epi::SPLIT || NSRC == 1, "a split contraction has one source");
    auto slice_begin = [&](int sl) { return (int)((uint32_t)ktiles * (uint32_t)sl / (uint32_t)p.ksplit); };

    auto tile_coords = [&](int i, int &batch, int &m0, int &n0) {
        int id = xcd * per_xcd + qx + i * wg_per_xcd;
        if (TAIL && i == my_whole) id = whole + piece / p.pieces;
        const int nt = id % tiles_n;
        id /= tiles_n;
        const int mt = id % tiles_m;
        batch = id / tiles_m;
        m0 = mt * BM;
        n0 = nt * BNS;
    };

    // the K steps of the cut tile, counted through the sources
    auto piece_begin = [&](int sl) { return __builtin_amdgcn_readfirstlane((int)((uint32_t)(ktiles * NSRC) * (uint32_t)sl / (uint32_t)p.pieces)); };
    // the cut tile's first K step: of source 1, or counted in source 0; steps in that source and, after it, in source 1
    struct Entry {
        int k0, left, left1;
        bool second;
    };
    auto enter_piece = [&]() -> Entry {
        const int sl = piece % p.pieces, k0 = piece_begin(sl), k1 = piece_begin(sl + 1);
        if (NSRC == 2 && k0 >= ktiles) return {k0 - ktiles, k1 - k0, 0, true};
        if (NSRC == 2 && k1 > ktiles) return {k0, ktiles - k0, k1 - ktiles, false};
        return {k0, k1 - k0, 0, false};
    };

    // ---- the two load streams.  A and B of a K step are fetched at different times, so each stream keeps
    // its own position: a wave-uniform pointer that advances by one K step, the K steps left in the current
    // source, and the lanes' byte offsets inside the tile (recomputed when a tile is entered, because an
    // edge tile clamps them).  All per-step work is a handful of scalar instructions: with one wave per
    // SIMD, whatever is issued between MFMAs and does not fit under them is lost matrix time (an earlier
    // version that derived the addresses of every load from the K step's number, i.e. from integer
    // divisions, spent more scalar instructions on them than the step has MFMA issue slots).
    const char *ptrA, *ptrB;
    int leftA, leftB, srcA = 0, srcB = 0, iA = 0, iB = 0;
    int left1A = ktiles, left1B = ktiles;   // K steps in the second source
    long bA = 0, bB = 0;     // byte offset of the current tile inside a source (second source: same offset)
    uint32_t offA[LA], offB[LB];
    const long kA = 2 * (A_MC ? (long)BK * p.lda[0] : (long)BK);
    const long kB = 2 * (B_NC ? (long)BK * p.ldb[0] : (long)BK);
    const int bset = (NSET == 2) ? wave / (TL::NW / 2) : 0;   // the first half of the waves fetches set 0

    auto enter_A = [&](int i) {
        int batch, m0, n0;
        tile_coords(i, batch, m0, n0);
        const int rem = p.M - m0;
#pragma unroll
        for (int q = 0; q < LA; ++q) {
            const int L = (wave * LA + q) * 64 + lane;   // LDS chunk position inside the operand tile
            if constexpr (A_MC) {
                constexpr int cpr = BM / 8;
                const int k = L / cpr, pc = L % cpr;
                int c = ((((pc >> 2) ^ ftr<BM>(k)) << 2) | (pc & 3)) << 3;
                c = c < rem ? c : rem - 8;
                offA[q] = 2u * ((uint32_t)k * (uint32_t)p.lda[0] + (uint32_t)c);
            } else {
                const int r = L >> 2, c = (L & 3) ^ fkc(r);
                const int rr = r < rem ? r : rem - 1;
                offA[q] = 2u * ((uint32_t)rr * (uint32_t)p.lda[0] + 8u * c);
            }
        }
        bA = 2 * ((long)batch * p.a_batch[0] + (A_MC ? (long)m0 : (long)m0 * p.lda[0]));
        ptrA = reinterpret_cast<const char *>(p.A[0]) + bA;
        if constexpr (NSRC == 2) bA = 2 * ((long)batch * p.a_batch[1] + (A_MC ? (long)m0 : (long)m0 * p.lda[0]));
        leftA = ktiles;
        srcA = 0;
        if constexpr (Epi::SPLIT) {
            const int sl = batch % p.ksplit, k0 = slice_begin(sl);
            ptrA = reinterpret_cast<const char *>(p.A[0]) + kA * k0 +
                   2 * ((long)(batch / p.ksplit) * p.a_batch[0] + (A_MC ? (long)m0 : (long)m0 * p.lda[0]));
            leftA = slice_begin(sl + 1) - k0;
        }
        if constexpr (TAIL)
            if (i == my_whole) {
                const Entry e = enter_piece();
                if (NSRC == 2 && e.second) ptrA = reinterpret_cast<const char *>(p.A[NSRC - 1]) + bA;
                ptrA += kA * e.k0;
                leftA = e.left;
                left1A = e.left1;
                if (NSRC == 2 && e.left1 == 0) srcA = 1;   // nothing left in the second source
            }
    };
    auto enter_B = [&](int i) {
        int batch, m0, n0;
        tile_coords(i, batch, m0, n0);
        const int rem = p.N - n0;
#pragma unroll
        for (int q = 0; q < LB; ++q) {
            const int L = ((wave * LB + q) * 64 + lane) & (TL::BN * 4 / NSET - 1);
            if constexpr (B_NC) {
                constexpr int cpr = BNS / 8;
                const int k = L / cpr, pc = L % cpr;
                int c = ((((pc >> 2) ^ ftr<BNS>(k)) << 2) | (pc & 3)) << 3;
                c = c < rem ? c : rem - 8;
                offB[q] = 2u * ((uint32_t)k * (uint32_t)p.ldb[0] + (uint32_t)c);
            } else {
                const int r = L >> 2, c = (L & 3) ^ fkc(r);
                const int rr = r < rem ? r : rem - 1;
                offB[q] = 2u * ((uint32_t)rr * (uint32_t)p.ldb[0] + 8u * c);
            }
        }
        if constexpr (!Epi::SPLIT) {
            // a scalar load: a vector load would count among the ring's
            typedef const __attribute__((address_space(4))) int32_t *const_ptr;
            if (p.b_map) batch = ((const_ptr)p.b_map)[batch];
        }
        const long in_b = B_NC ? (long)n0 : (long)n0 * p.ldb[0];
        const int s = (NSET == 2) ? bset : 0;
        ptrB = reinterpret_cast<const char *>(s ? p.B[1] : p.B[0]) + 2 * ((long)batch * (s ? p.b_batch[1] : p.b_batch[0]) + in_b);
        if constexpr (NSRC == 2) bB = 2 * ((long)batch * p.b_batch[1] + in_b);
        leftB = ktiles;
        srcB = 0;
        if constexpr (Epi::SPLIT) {
            const int sl = batch % p.ksplit, k0 = slice_begin(sl);
            ptrB = reinterpret_cast<const char *>(s ? p.B[1] : p.B[0]) + kB * k0 +
                   2 * ((long)(batch / p.ksplit) * (s ? p.b_batch[1] : p.b_batch[0]) + in_b);
            leftB = slice_begin(sl + 1) - k0;
        }
        if constexpr (TAIL)
            if (i == my_whole) {
                const Entry e = enter_piece();
                if (NSRC == 2 && e.second) ptrB = reinterpret_cast<const char *>(p.B[NSRC - 1]) + bB;
                ptrB += kB * e.k0;
                leftB = e.left;
                left1B = e.left1;
                if (NSRC == 2 && e.left1 == 0) srcB = 1;   // nothing left in the second source
            }
    };
    // One K step further.  Past the end of the stream the last K step is fetched again, into slots nobody
    // reads, so that the wait counts below always hold.
    auto advance_A = [&]() {
        ptrA += kA;
        if (--leftA == 0) {
            if (NSRC == 2 && srcA == 0) {
                srcA = 1;
                ptrA = reinterpret_cast<const char *>(p.A[1]) + bA;
                leftA = left1A;
            } else if (iA + 1 < my_tiles) {
                enter_A(++iA);
            } else {
                ptrA -= kA;
                leftA = 1;
            }
        }
    };
    auto advance_B = [&]() {
        ptrB += kB;
        if (--leftB == 0) {
            if (NSRC == 2 && srcB == 0) {
                srcB = 1;
                ptrB = reinterpret_cast<const char *>(p.B[1]) + bB;
                leftB = left1B;
            } else if (iB + 1 < my_tiles) {
                enter_B(++iB);
            } else {
                ptrB -= kB;
                leftB = 1;
            }
        }
    };
    const uint32_t ldsA = lds0 + wave * (LA * 1024);
    const uint32_t ldsB = lds0 + TL::a_bytes + wave * (LB * 1024);
    auto issue_A = [&](uint32_t slot, int i) { dma16s(TAIL ? uniform(ptrA) : ptrA, offA[i], ldsA + slot + i * 1024); };
    auto issue_B = [&](uint32_t slot, int j) { dma16s(TAIL ? uniform(ptrB) : ptrB, offB[j], ldsB + slot + j * 1024); };
    auto next_slot = [&](uint32_t s) -> uint32_t { return s + TL::stage == TL::ring ? 0u : s + TL::stage; };

    f32x16 acc[NSET][MI][NI];
    auto zero_acc = [&]() {
#pragma unroll
        for (int s = 0; s < NSET; ++s)
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[s][i][j][r] = 0.f;
    };

    enter_A(0);
    enter_B(0);
#pragma unroll
    for (int g = 0; g < S; ++g) {  // the whole ring: K steps 0 .. S-1
#pragma unroll
        for (int i = 0; i < LA; ++i) issue_A(g * TL::stage, i);
#pragma unroll
        for (int j = 0; j < LB; ++j) issue_B(g * TL::stage, j);
        advance_A();
        advance_B();
    }

    // LDS offsets of the lane's fragments inside a stage.  KC: one per 16-wide slice, blocks 2 KB apart.
    // K-slow: one per block, slices 16 rows apart.
    constexpr int NFA = A_MC ? MI : 2, NFB = B_NC ? NI : 2;
    int fragA[NFA], fragB[NFB];
    {
        const int g16 = lane >> 4, r = lane & 15, krow = 8 * (g16 >> 1) + (r >> 2);
#pragma unroll
        for (int f = 0; f < NFA; ++f) {
            if constexpr (A_MC) {
                const int co = (wm0 + f * 32 + 16 * (g16 & 1) + 4 * (r & 3)) * 2;
                fragA[f] = krow * (BM * 2) + ((((co >> 6) ^ ftr<BM>(krow)) << 6) | (co & 63));
            } else {
                const int row = wm0 + (lane & 31);
                fragA[f] = row * 64 + (((2 * f + (lane >> 5)) ^ fkc(lane & 31)) << 4);
            }
        }
#pragma unroll
        for (int f = 0; f < NFB; ++f) {
            if constexpr (B_NC) {
                const int co = (wn0 + f * 32 + 16 * (g16 & 1) + 4 * (r & 3)) * 2;
                fragB[f] = TL::a_bytes + krow * (BNS * 2) + ((((co >> 6) ^ ftr<BNS>(krow)) << 6) | (co & 63));
            } else {
                const int row = wn0 + (lane & 31);
                fragB[f] = TL::a_bytes + row * 64 + (((2 * f + (lane >> 5)) ^ fkc(lane & 31)) << 4);
            }
        }
    }
    // Fragments of a 16-wide K slice in the order their first MFMA needs them: A block 0, the B
    // blocks (counted through the operand sets), A blocks 1 ..
    constexpr int NF = MI + NB;
    auto load_frag = [&](uint32_t slot, int kk, int f, bf16x8 (&af)[MI], bf16x8 (&bfr)[NB]) {
        const char *la = smem + slot;
        if (f == 0 || f > NB) {
            const int i = f == 0 ? 0 : f - NB;
            if constexpr (A_MC)
                af[i] = frag_tr(la + fragA[i % NFA] + kk * 16 * (BM * 2), 4 * BM * 2);
            else
                af[i] = *reinterpret_cast<const bf16x8 *>(la + fragA[kk] + i * 2048);
        } else {
            const int q = f - 1, s = q / NI, j = q % NI;
            if constexpr (B_NC)
                bfr[q] = frag_tr(la + fragB[j % NFB] + s * BSET_BYTES + kk * 16 * (BNS * 2), 4 * BNS * 2);
            else
                bfr[q] = *reinterpret_cast<const bf16x8 *>(la + fragB[kk] + s * BSET_BYTES + j * 2048);
        }
    };

    // The MI * NB MFMAs of a K slice are issued one per "slot"; the first slots also carry the LDS fragment
    // reads of the next slice, and some this wave's direct loads for the ring, so that those issue in
    // the shadow of the matrix pipe and the fragments have arrived when the slice ends.  Where B streams K-slow rows
    // and A is K-contiguous (gate/up and down, forward) the loads of eight waves are spread over the slice from its
    // first slot: gate/up of 64 segments of 256 tokens at d = 2048, d_ff = 5632 792 -> 779 us, down of 128 at d = 1024
    // 257 -> 242.  Elsewhere they stay in the second half (dX of the first shape, two K-contiguous sources: 749, spread
    // 762; down of 16 segments of 448 at d = 1280 on four waves: 76, spread 78).  Fragments are
    // double buffered in registers.  The single barrier of a K step sits between its two slices: by then
    // every wave has finished reading step g-1 (its ring slot may be refilled with step g+S-1) and step
    // g+1 has landed for everyone (its first slice can be fetched behind the second slice's MFMAs).
    constexpr int NM = NB * MI;
    auto load_slot = [](int l, int n) { return (B_NC && !A_MC && NSRC == 1 && TL::NW == 8) ? l * NM / n : NM / 2 + l * (NM / 2) / n; };
    bf16x8 a0[MI], b0[NB], a1[MI], b1[NB];
    wait_vmcnt<(S - 1) * (LA + LB)>();  // steps 1 .. S-1 may still be in flight
    ring_barrier();
#pragma unroll
    for (int f = 0; f < NF; ++f) load_frag(0, 0, f, a0, b0);

    uint32_t cur = 0, nxt = TL::stage;          // ring slots of step g and g+1
    uint32_t slotA = (S - 1) * TL::stage;       // slot of step g+S-1: the next one A refills
    // One K step g:
    //   first half:  A chunks of step g+S-1 (into the slot step g-1 left at the previous barrier)
    //   second half: B chunks of step g+S (into the slot step g itself left at this step's barrier:
    //                every wave has fetched its last fragments of step g by then)
    // The B operand is the one that streams from HBM, hence the longer lead.  Across a tile boundary the A
    // chunks that the next tile's first step would issue are issued half a step early, in the last step of
    // the tile, so that everything the next tile's first S-1 steps wait for is older than the epilogue's
    // stores: loads and stores share vmcnt and retire in order, and a wait may only leave younger
    // operations pending.  "All but the newest (S-2)(LA+LB) loads have landed" means "step g+1 is
    // complete".  extra: store instructions of the previous tile's epilogue that may still be pending.
    auto step = [&](auto first_c, auto last_c, int extra) {
        constexpr bool first = decltype(first_c)::value, last = decltype(last_c)::value;
        constexpr int kWait = (S - 2) * (LA + LB);
#pragma unroll
        for (int sl = 0; sl < NM; ++sl) {
            const int i = sl / NB, q = sl % NB;
            acc[q / NI][i][q % NI] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b0[q], a0[i], acc[q / NI][i][q % NI], 0, 0, 0);
#pragma unroll
            for (int f = 0; f < NF; ++f)
                if (f * NM / (2 * NF) == sl) load_frag(cur, 1, f, a1, b1);
            if constexpr (!first) {
#pragma unroll
                for (int l = 0; l < LA; ++l)
                    if (load_slot(l, LA) == sl) issue_A(slotA, l);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (!first) advance_A();
        if (extra >= 32)
            wait_vmcnt<kWait + 32>();
        else if (extra >= 16)
            wait_vmcnt<kWait + 16>();
        else
            wait_vmcnt<kWait>();
        ring_barrier();
#pragma unroll
        for (int sl = 0; sl < NM; ++sl) {
            const int i = sl / NB, q = sl % NB;
            acc[q / NI][i][q % NI] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b1[q], a1[i], acc[q / NI][i][q % NI], 0, 0, 0);
#pragma unroll
            for (int f = 0; f < NF; ++f)
                if (f * NM / (2 * NF) == sl) load_frag(nxt, 0, f, a0, b0);
#pragma unroll
            for (int l = 0; l < LB; ++l)
                if (load_slot(l, LB) == sl) issue_B(cur, l);
            if constexpr (last) {
#pragma unroll
                for (int l = 0; l < LA; ++l)
                    if (load_slot(l, LA) == sl) issue_A(cur, l);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        advance_B();
        if constexpr (last) advance_A();
        slotA = cur;
        cur = nxt;
        nxt = next_slot(nxt);
    };

    // Epilogue of one tile, wave-local: the wave's WM x WN sub-tile leaves in blocks of 32 rows
    // through the wave's own staging area (XOR-swizzled 16-byte chunks), as 16-byte stores that
    // are contiguous along n.  Accumulator element r of a 32x32 block is row m = lane & 31,
    // column n = 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3).  Edge tiles (not full) mask the rows and chunks
    // beyond the matrix.
    char *stg = smem + TL::ring + wave * TL::stage_out;
    constexpr int JG = TL::JG < NI ? TL::JG : NI;   // 32-column blocks staged at a time
    constexpr int CP = JG * 4;             // 16-byte chunks per staged row
    auto epilogue = [&](auto full_c, int batch, int m0, int n0) {
        constexpr bool full = decltype(full_c)::value;
        // keeps the two instances apart: merged, their common part would hold every packed value at once
        if constexpr (full)
            asm volatile("; interior tile" ::: "memory");
        else
            asm volatile("; edge tile" ::: "memory");
        int el = lane;
        asm volatile("" : "+v"(el));   // lane constants of the epilogue are formed here, not kept across the K loop
        const int r = el & 31, h = el >> 5;
        if constexpr (Epi::SPLIT) {
            // fp32 partial sums straight from the accumulators: 16 bytes per lane, 128 bytes of a row over
            // four stores
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                const int m = m0 + wm0 + i * 32 + r;
#pragma unroll
                for (int s = 0; s < NSET; ++s)
#pragma unroll
                    for (int j = 0; j < NI; ++j)
#pragma unroll
                        for (int rq = 0; rq < 4; ++rq) {
                            const int n = n0 + wn0 + j * 32 + 8 * rq + 4 * h;
                            if (full || (m < p.M && n < p.N))
                                *reinterpret_cast<float4 *>(epi.part(s, batch, m, n)) =
                                    make_float4(acc[s][i][j][rq * 4 + 0], acc[s][i][j][rq * 4 + 1],
                                                acc[s][i][j][rq * 4 + 2], acc[s][i][j][rq * 4 + 3]);
                        }
            }
            return;
        }
        // The lane's position in the stores: row lane / CP of every RPI rows, chunk lane % CP.  The
        // address of every plane is a running pointer.
        constexpr int RPI = 64 / CP;
        const int srow = el / CP, sc = el % CP;
        const int ncol = n0 + wn0 + sc * 8;
        const long step_bytes = (long)RPI * epi.row_bytes();
        char *out[Epi::NOUT];
#pragma unroll
        for (int o = 0; o < Epi::NOUT; ++o)
            if (epi.enabled(o)) out[o] = reinterpret_cast<char *>(epi.ptr(o, batch, m0 + wm0 + srow, ncol));
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int mb = m0 + wm0 + i * 32;
            // all planes of one 32-row block before the next block: its accumulators are read
            // into registers once
#pragma unroll
            for (int o = 0; o < Epi::NOUT; ++o) {
                if (!epi.enabled(o)) continue;
                char *dst = out[o];
#pragma unroll
                for (int jg = 0; jg < NI; jg += JG) {
#pragma unroll
                    for (int jj = 0; jj < JG; ++jj)
#pragma unroll
                        for (int rq = 0; rq < 4; ++rq) {
                            const int j = jg + jj;
                            float v[NSET][4];
#pragma unroll
                            for (int s = 0; s < NSET; ++s)
#pragma unroll
                                for (int e = 0; e < 4; ++e) v[s][e] = acc[s][i][j][rq * 4 + e];
                            const u32x2 pk = epi.pack(o, v);
                            const int c = jj * 4 + rq;
                            *reinterpret_cast<u32x2 *>(stg + r * (CP * 16) + ((c ^ (r & (CP - 1))) << 4) + h * 8) = pk;
                            __builtin_amdgcn_sched_barrier(0);  // one quad at a time: keeps register use flat
                        }
                    __builtin_amdgcn_wave_barrier();
                    dst = out[o] + jg * 64;
#pragma unroll
                    for (int it = 0; it < 32 / RPI; ++it) {
                        const int row = it * RPI + srow;
                        const u32x4 val = *reinterpret_cast<const u32x4 *>(stg + row * (CP * 16) + ((sc ^ (row & (CP - 1))) << 4));
                        // streamed output: non-temporal, so that it does not push the operands that later
                        // tiles share (activations of the segment) out of the caches
                        if (full || (mb + row < p.M && ncol + jg * 32 < p.N))
                            __builtin_nontemporal_store(val, reinterpret_cast<u32x4 *>(dst));
                        dst += step_bytes;
                        asm volatile("" : "+v"(dst));
                    }
                    __builtin_amdgcn_wave_barrier();
                }
                out[o] = dst - (NI - JG) * 64;
            }
        }
    };

    // 16-byte store instructions a wave issues per interior tile
    int nst = Epi::SPLIT ? MI * NB * 4 : 0;
#pragma unroll
    for (int o = 0; o < Epi::NOUT; ++o)
        if (epi.enabled(o)) nst += MI * NI * 2;
    using T = std::true_type;
    using F = std::false_type;
    int extra = 0;
    for (int tile_i = 0; tile_i < my_tiles; ++tile_i) {
        zero_acc();
        int batch, m0, n0;
        tile_coords(tile_i, batch, m0, n0);
        int total = ktiles * NSRC;
        if constexpr (Epi::SPLIT) total = slice_begin(batch % p.ksplit + 1) - slice_begin(batch % p.ksplit);
        if (TAIL && tile_i == my_whole) total = piece_begin(piece % p.pieces + 1) - piece_begin(piece % p.pieces);
        // the first S-1 K steps of a tile run while the previous tile's stores drain
        step(T(), F(), extra);
        for (int t = 1; t < total - 1; ++t) step(F(), F(), t < S - 1 ? extra : 0);
        step(F(), T(), total - 1 < S - 1 ? extra : 0);
        if constexpr (TAIL)
            if (tile_i == my_whole) {
                // accumulators as they lie, 1 KB per store; rows and columns beyond the matrix are never read
                asm volatile("; piece" ::: "memory");
                int el = lane;
                asm volatile("" : "+v"(el));
                char *dst = reinterpret_cast<char *>(p.tail) + ((size_t)piece * TL::NW + wave) * (MI * NB * 4 * 1024);
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int j = 0; j < NI; ++j)
#pragma unroll
                        for (int s = 0; s < NSET; ++s)
#pragma unroll
                            for (int rq = 0; rq < 4; ++rq) {
                                *reinterpret_cast<float4 *>(dst + (uint32_t)el * 16u) =
                                    make_float4(acc[s][i][j][rq * 4 + 0], acc[s][i][j][rq * 4 + 1],
                                                acc[s][i][j][rq * 4 + 2], acc[s][i][j][rq * 4 + 3]);
                                dst += 1024;
                                __builtin_amdgcn_sched_barrier(0);
                            }
                break;   // a workgroup's last tile
            }
        if (m0 + BM <= p.M && n0 + BNS <= p.N) {
            epilogue(T(), batch, m0, n0);
            extra = nst;
        } else {
            epilogue(F(), batch, m0, n0);
            extra = 0;   // masked stores may not have been issued: wait as if there were none
        }
    }
    wait_vmcnt<0>();  // no direct load may still be writing LDS when the workgroup retires
}

// Adds the K slices of the cut tiles in slice order and runs the epilogue on the sums.  A wavefront takes 32 rows x 64
// columns (of every set) of a wavefront of the GEMM; they leave through LDS as whole lines, like an interior tile's.
// Bound by reading the sums back (256 KB a slice, 256-row tile), which sit in the memory-side cache.
template <int NSET, class TL, class Epi>
__global__ __launch_bounds__(256) void tail_kernel(const Params p, const Epi epi, int whole, int jobs)
{
    constexpr int MI = TL::MI, NI = TL::NB / NSET, BNS = TL::BN / NSET, JG = 2;
    static_assert(NI % JG == 0, "blocks of 64 columns");
    constexpr int CP = JG * 4, RPI = 64 / CP;
    __shared__ __attribute__((aligned(16))) char stage[4][32 * CP * 16];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int job = blockIdx.x * 4 + wv;
    if (job >= jobs) return;
    const int jg = job % (NI / JG) * JG;
    job /= NI / JG;
    const int i = job % MI;
    job /= MI;
    const int wave = job % TL::NW, t = job / TL::NW;
    const int tiles_n = (p.N + BNS - 1) / BNS, tiles_m = (p.M + TL::BM - 1) / TL::BM;
    int id = whole + t;
    const int n0 = id % tiles_n * BNS + wave % TL::WNV * (NI * 32) + jg * 32;
    id /= tiles_n;
    const int m0 = id % tiles_m * TL::BM + wave / TL::WNV * (MI * 32) + i * 32, batch = id / tiles_m;

    constexpr int Q = JG * NSET * 4;   // quads of a lane
    float4 v[Q];
    const size_t pitch = (size_t)TL::NW * (MI * TL::NB * 4 * 64);
    const float4 *src = reinterpret_cast<const float4 *>(p.tail) + (size_t)t * p.pieces * pitch +
                        (size_t)wave * (MI * TL::NB * 4 * 64) + (i * NI + jg) * (NSET * 4 * 64) + lane;
#pragma unroll
    for (int q = 0; q < Q; ++q) v[q] = src[q * 64];
#pragma unroll 2
    for (int s = 1; s < p.pieces; ++s) {
        src += pitch;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const float4 a = src[q * 64];
            v[q].x += a.x; v[q].y += a.y; v[q].z += a.z; v[q].w += a.w;
        }
    }
    const int r = lane & 31, h = lane >> 5, srow = lane / CP, sc = lane % CP;
    char *stg = stage[wv];
#pragma unroll
    for (int o = 0; o < Epi::NOUT; ++o) {
        if (!epi.enabled(o)) continue;
#pragma unroll
        for (int jj = 0; jj < JG; ++jj)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                float x[NSET][4];
#pragma unroll
                for (int s = 0; s < NSET; ++s) {
                    const float4 a = v[(jj * NSET + s) * 4 + rq];
                    x[s][0] = a.x; x[s][1] = a.y; x[s][2] = a.z; x[s][3] = a.w;
                }
                const u32x2 pk = epi.pack(o, x);
                *reinterpret_cast<u32x2 *>(stg + r * (CP * 16) + (((jj * 4 + rq) ^ (r & (CP - 1))) << 4) + h * 8) = pk;
            }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int it = 0; it < 32 / RPI; ++it) {
            const int row = it * RPI + srow;
            const u32x4 val = *reinterpret_cast<const u32x4 *>(stg + row * (CP * 16) + ((sc ^ (row & (CP - 1))) << 4));
            if (m0 + row < p.M && n0 + sc * 8 < p.N)
                *reinterpret_cast<u32x4 *>(epi.ptr(o, batch, m0 + row, n0 + sc * 8)) = val;
        }
        __builtin_amdgcn_wave_barrier();
    }
}

inline int cu_count()
{
    static int n = 0;
    if (n == 0) {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 8)
            return 256;   // not kept: a later call may find the device
        n = cus / 8 * 8;
    }
    return n;
}

inline int persistent_grid() { return cu_count(); }

template <int NSET, int NSRC, bool A_MC, bool B_NC, class TL, class Epi, bool TAIL = false>
inline hipError_t launch(const Params &p, const Epi &epi, hipStream_t st)
{
    if (p.K % BK != 0 || p.K < 2 * BK || p.N % 8 != 0 || p.M < 1 || p.N < 8 || (A_MC && p.M % 8 != 0)) return hipErrorInvalidValue;
    if (NSRC == 2 && (p.lda[0] != p.lda[1] || p.ldb[0] != p.ldb[1])) return hipErrorInvalidValue;
    if (NSET == 2 && p.ldb[0] != p.ldb[1]) return hipErrorInvalidValue;
    if (Epi::SPLIT && (p.ksplit < 1 || p.ksplit > 1024 || p.K > kMaxCutK || p.batches % p.ksplit != 0 || p.K / BK < 2 * p.ksplit)) return hipErrorInvalidValue;
    const int cus = cu_count();
    auto kern = gemm2_kernel<NSET, NSRC, A_MC, B_NC, TAIL, TL, Epi>;
    static bool configured = false;  // per instantiation
    if (!configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, TL::total);
        if (e != hipSuccess) return e;
        configured = true;
    }
    constexpr int BNS = TL::BN / NSET;
    const long ntiles = (long)p.batches * ((p.M + TL::BM - 1) / TL::BM) * ((p.N + BNS - 1) / BNS);
    long blocks = (ntiles + 7) / 8 * 8;
    if (blocks > cus) blocks = cus;  // every workgroup walks several tiles
    if (TAIL) {
        if (p.pieces < 1 || !p.tail || ntiles % cus == 0 || ntiles % cus * p.pieces > cus || p.K / BK * NSRC < 2 * p.pieces ||
            p.tail_floats < (size_t)(ntiles % cus) * p.pieces * TL::BM * TL::BN || p.K > kMaxCutK || ntiles >= (1L << 31))
            return hipErrorInvalidValue;
        blocks = cus;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(TL::threads), TL::total, st, p, epi);
    if constexpr (TAIL) {
        const long cut = ntiles % cus;
        const int jobs = (int)(cut * TL::NW * TL::MI * (TL::NB / NSET / 2));
        hipLaunchKernelGGL((tail_kernel<NSET, TL, Epi>), dim3((unsigned)((jobs + 3) / 4)), dim3(256), 0, st, p, epi,
                           (int)(ntiles - cut), jobs);
    }
    return hipGetLastError();
}

// Tile shapes in use.  Eight waves (two per SIMD) where the tile is 256 rows tall: with four waves of
// 128 x 128 the CU's vector-memory path delivered 16 bytes per cycle at one wave per SIMD, and weight
// gradients (short contractions) waited for their own epilogues.  Sustained rates on N(0,1) data,
// TFLOP/s, four-wave kernel -> this one: X_s^T dG_s of 64 segments of 256 tokens at d = 2048, d_ff = 5632:
// 695 -> 860; dY Wd_bar^T of the same: 840 -> 930; a single 8192^3 product: 1300, where the chip is at
// its power limit.  192 rows need four waves (12 KB of A do not divide by eight); 128 rows ran faster
// with four waves and three stages than with eight and four (A Wd_bar of 32 segments at d = 1024: 45
// against 53 us).
using T256 = Tile<2, 4, 4, 2, 4>;
// Two operand sets: a wave of T256 would own 32 columns of each and store 64 bytes of a row, half a line; 64 x 64 per
// wave and set stores whole lines.  Gate/up with G and U saved, us: 64 segments of 256 tokens at d = 2048, d_ff = 5632
// 852 -> 824; 128 segments at d = 1024, d_ff = 2816 491 -> 467; 8 of 1024 at d = 2048 425 -> 408.  The activation alone
// (half the stores): 803 -> 799, 443 -> 438, 400 -> 397.
using T256x2 = Tile<4, 2, 2, 4, 4>;
using T192 = Tile<2, 2, 3, 4, 4>;
using T128 = Tile<2, 2, 2, 4, 3>;
using T64 = Tile<2, 2, 1, 4, 4>;
using W128 = Tile<2, 4, 2, 2, 4>;   // 128 rows of a weight gradient

// Rounds of tiles over the CUs, in units of the time of one round.
inline double rounds_of(const Params &p, int bm, int bns)
{
    const long tiles = (long)p.batches * ((p.M + bm - 1) / bm) * ((p.N + bns - 1) / bns);
    return (double)((tiles + cu_count() - 1) / cu_count());
}

// Time of a tile's K step, us, all CUs busy on slabs of T = 64 .. 1024 rows.
constexpr double step_us(int rows) { return rows == 256 ? 0.90 : rows == 192 ? 0.72 : rows == 128 ? 0.62 : 0.42; }

// Tile height of a contraction whose rows are the tokens of a segment: the shortest estimated time, rounds of tiles
// over the CUs times the time of a step.  A taller tile costs less per row, a lower one wastes fewer rows of a segment
// and fewer CUs of the last round.  128 rows of a 256-row segment read the merged operand twice: 64 segments, K = 4096,
// N = 1536 take 297 us in two rounds of 256 rows and 317 in three of 128 (dX of the same 527 and 593), 32 segments,
// K = 2816, N = 1024 94 in half a round of 256 and 67 in one of 128.
struct Form {
    int rows;
    int pieces;   // K slices of a tile of the last round, 0 where it is not cut
};

inline size_t tail_floats(const Params &p, const Form &f, int bns)
{
    const long tiles = (long)p.batches * ((p.M + f.rows - 1) / f.rows) * ((p.N + bns - 1) / bns);
    return (size_t)(tiles % cu_count()) * f.pieces * f.rows * 256;
}

// With scratch for its partial sums (p.tail) a last round that leaves CUs without a tile may be cut over K, one slice for
// each CU: it costs its share of the steps, the sums a CU writes (45 KB a us) and a launch that adds them (4.5 us and
// the rate of the memory-side cache).  A form has to promise 3 % more than the best one before it, in the order of falling
// tile heights and rising slices: the promise of more slices is kept in part only (the cheapest estimate of all instead:
// 5 x 1655 rows at d = 384, d_ff = 1728 88 -> 96 us, 4 x 704 at 1472, 3200 121 -> 124, 4 x 1024 at 2048, 5632 268 -> 272).
inline Form plan_form(const Params &p, int bns, int nsrc, size_t floats)
{
    const int cus = cu_count(), steps = p.K / BK * nsrc;
    Form best = {256, 0};
    double best_t = 0;
    for (int rows = 256; rows >= 64; rows -= 64) {
        const double us = step_us(rows);
        const double t = us * steps * rounds_of(p, rows, bns);
        if (rows == 256 || t < best_t) {
            best = {rows, 0};
            best_t = t;
        }
        const long tiles = (long)p.batches * ((p.M + rows - 1) / rows) * ((p.N + bns - 1) / bns), cut = tiles % cus;
        if (!p.tail || cut == 0 || p.K > kMaxCutK || tiles >= (1L << 31)) continue;
        const double kb = rows * 256 * 4 / 1000.0;
        for (int n = 2; cut * n <= cus && 4 * n <= steps && (size_t)(cut * n) * rows * 256 <= floats; ++n) {
            const double c = us * (steps * (double)(tiles / cus) + (steps + n - 1) / n + 2) + kb / 45.0 + 4.5 + cut * n * kb / 4000.0;
            if (c < 0.97 * best_t) {
                best = {rows, n};
                best_t = c;
            }
        }
    }
    return best;
}

// The form of unlimited scratch where the scratch holds it, so that a caller who sizes its scratch from that form gets it
// and more scratch changes nothing; else one that fits.
inline Form tile_form(const Params &p, int bns, int nsrc)
{
    const Form f = plan_form(p, bns, nsrc, (size_t)-1);
    return f.pieces && tail_floats(p, f, bns) > p.tail_floats ? plan_form(p, bns, nsrc, p.tail_floats) : f;
}

inline int tile_rows(const Params &p, int bns)
{
    Params q = p;
    q.K = BK;   // the rounds alone decide
    q.tail = nullptr;
    return tile_form(q, bns, 1).rows;
}

template <int NSET, int NSRC, bool A_MC, bool B_NC, class Epi, bool TAIL>
inline hipError_t launch_tile(int rows, const Params &p, const Epi &e, hipStream_t st)
{
    switch (rows) {
    case 256: return launch<NSET, NSRC, A_MC, B_NC, std::conditional_t<NSET == 2, T256x2, T256>, Epi, TAIL>(p, e, st);
    case 192: return launch<NSET, NSRC, A_MC, B_NC, T192, Epi, TAIL>(p, e, st);
    case 128: return launch<NSET, NSRC, A_MC, B_NC, T128, Epi, TAIL>(p, e, st);
    default: return launch<NSET, NSRC, A_MC, B_NC, T64, Epi, TAIL>(p, e, st);
    }
}

template <int NSET, int NSRC, bool A_MC, bool B_NC, class Epi>
inline hipError_t launch_rows(const Params &p0, const Epi &e, hipStream_t st)
{
    const Form f = tile_form(p0, 256 / NSET, NSRC);
    // an instance of its own for the cut round: its code costs every launch 1 .. 2 us
    if constexpr (Epi::TAIL) {
        if (f.pieces) {
            Params p = p0;
            p.pieces = f.pieces;
            return launch_tile<NSET, NSRC, A_MC, B_NC, Epi, true>(f.rows, p, e, st);
        }
    }
    return launch_tile<NSET, NSRC, A_MC, B_NC, Epi, false>(f.rows, p0, e, st);
}

// Tile of a weight gradient (K = tokens of a segment): both heights take the same time per element
// (bound by their stores), so the one that wastes less of the last round.
template <int NSET, int NSRC, bool A_MC, bool B_NC, class Epi>
inline hipError_t launch_weight(const Params &p, const Epi &e, hipStream_t st)
{
    if (rounds_of(p, 256, 256) <= 0.51 * rounds_of(p, 128, 256)) return launch<NSET, NSRC, A_MC, B_NC, T256>(p, e, st);
    return launch<NSET, NSRC, A_MC, B_NC, W128>(p, e, st);
}

}  // namespace gemm2
}  // namespace lory
