// fp32 instantiation of the merged FFN (paper Eq. 1 / Eq. 2, SwiGLU experts)
// and of its backward, for arbitrary shapes at fp32 accuracy (rel-L2 <= 1e-5).
//
// Every stage is a small dense contraction - the merge is w [S,E] x stack [E,n] (with few experts or segments a
// kernel of its own that streams the stack), the scatter w^T [E,S] x slab [S,n], the inner products slab [S,n] x stack^T [n,E], the rest are the layer's token
// GEMMs - so one kernel on the fp32 matrix instruction (v_mfma_f32_32x32x2_f32, full fp32 products and
// sums) runs them all, and independent ones share a launch: the shapes of this configuration are small and
// a pass is bound by the number of dependent launches (B=2, L=512, T=128, d=64, d_ff=256, E=4: 27 launches
// of 4-30 us each took 325 us per training step, 12 launches take 70 us; B=8, L=1024, T=256, d=256, d_ff=640,
// E=16: 1787 -> 616 us, 42 TFLOP/s).  SwiGLU and its derivative
// are epilogues.  Merged weights of a chunk of segments live in a workspace slab, so that the workspace
// stays bounded.
#include "lory_internal.h"

namespace lory {

namespace k {
hipError_t launch_dw_reduce(hipStream_t st, const float *partials, int slots, int rows, int cols, float *dw, int S,
                            int E);
}

namespace {

constexpr size_t kF32ChunkBudget = (size_t)512 << 20;  // workspace target per chunk of segments

// ---------------------------------------------------------------- the contraction kernel

typedef float f32x16 __attribute__((ext_vector_type(16)));

enum Mode { kStore = 0, kGateUp = 1, kGradAct = 2 };

// C_b[m][n] (+)= sum over sources q, k of A_{q,b}(m,k) * B_{q,b}(k,n); operand element (i,k) at
// base + i * s_i + k * s_k, one of the two strides being 1.
struct Problem {
    const float *A[2], *B[2];   // second source, or NULL; kGateUp: B[1] is the up projection's operand
    long a_batch, b_batch;      // elements between batch items
    long sAm, sAk, sBn, sBk;
    float *C;
    long c_batch;
    long ldc;
    long M, N, K;
    int batches;
    int ksplit;                 // slices of K; slice j writes C + j * c_slice
    long c_slice;
    int add;
    int vecA, vecB;             // 16-byte loads along k are aligned
    int split_waves;            // the four wavefronts share a 32 x 32 block (else a 64 x 64 tile)
    int blocks;                 // workgroups of this problem
};

constexpr int kMaxProblems = 7;
constexpr long kMaxGrid = (1L << 24) - 1;
struct Group {
    Problem p[kMaxProblems];
    int n;
    int first;                  // of this launch's workgroups, counted through the problems
};

// Elementwise operands of the epilogues, all with the layout of C.
struct Elementwise {
    float *U, *A;               // kGateUp: C receives G
    const float *G_in, *U_in;   // kGradAct: C receives dG
    float *dU;
};

constexpr int TK = 32;   // contraction indices of a step

__device__ inline float sigmoidf_(float z) { return 1.0f / (1.0f + expf(-z)); }

// One lane's share of 32 rows x 32 contraction indices of an operand, straight from memory: row lane & 31,
// indices 8 j + 4 (lane >> 5) + e for j, e = 0..3 (the matrix instruction pairs element (j, e) of both lane
// halves; any order does as long as A and B agree).  base: element (row of the lane, index 4 (lane >> 5) of the
// step); left: indices left from there (elements beyond are zero); rows: 16-byte loads along k are possible.
__device__ __forceinline__ void load_frag(float (&v)[16], const float *base, long s_k, int left, bool rows)
{
    if (rows && left >= TK - 4) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float4 f = *reinterpret_cast<const float4 *>(base + 8 * j);
            v[4 * j] = f.x; v[4 * j + 1] = f.y; v[4 * j + 2] = f.z; v[4 * j + 3] = f.w;
        }
    } else {
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int k = 8 * (q >> 2) + (q & 3);
            v[q] = 0.f;
            if (k < left) v[q] = base[k * s_k];
        }
    }
}

// 256 threads = 4 wavefronts of one 32 x 32 block (two in kGateUp: both operand sets share A).  Operands go
// straight from memory to the matrix instruction, one step ahead: no barrier in the loop, and a short
// contraction costs one memory latency.  p.split_waves: the wavefronts share one block and take a quarter
// of its steps each, added in LDS (few blocks); else they form a 64 x 64 tile.
template <int MODE>
__global__ __launch_bounds__(256) void contract_kernel(const Group grp, const Elementwise ew)
{
    constexpr int NSET = MODE == kGateUp ? 2 : 1;
    __shared__ float red[3][NSET][16][64];
    int bid = grp.first + blockIdx.x, pi = 0;
    while (bid >= grp.p[pi].blocks) bid -= grp.p[pi++].blocks;
    const Problem &p = grp.p[pi];
    const int tile = p.split_waves ? 32 : 64;
    const int tiles_n = (int)((p.N + tile - 1) / tile), tiles_m = (int)((p.M + tile - 1) / tile);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l31 = lane & 31, lh = lane >> 5;
    long n0 = (long)(bid % tiles_n) * tile;
    bid /= tiles_n;
    long m0 = (long)(bid % tiles_m) * tile;
    bid /= tiles_m;
    const int sl = bid % p.ksplit, b = bid / p.ksplit;
    const long steps_all = (p.K + TK - 1) / TK;
    int kb = (int)(steps_all * sl / p.ksplit), ke = (int)(steps_all * (sl + 1) / p.ksplit);
    const int nsrc = (MODE != kGateUp && p.A[1]) ? 2 : 1;
    int per_src = ke - kb, t0 = 0, t1 = per_src * nsrc;
    if (p.split_waves) {
        const int t = t1;
        t0 = t * wave / 4;
        t1 = t * (wave + 1) / 4;
    } else {
        m0 += (wave >> 1) * 32;
        n0 += (wave & 1) * 32;
        if (m0 >= p.M || n0 >= p.N) return;   // no barrier follows in this form
    }

    // rows and columns beyond the matrix repeat the last one; their results are not stored
    const long mrow = m0 + l31 < p.M ? m0 + l31 : p.M - 1, ncol = n0 + l31 < p.N ? n0 + l31 : p.N - 1;
    const long offA = b * p.a_batch + mrow * p.sAm + 4 * lh * p.sAk, offB = b * p.b_batch + ncol * p.sBn + 4 * lh * p.sBk;
    const bool rowsA = p.vecA && p.sAk == 1, rowsB = p.vecB && p.sBk == 1;
    f32x16 acc[NSET];
#pragma unroll
    for (int s = 0; s < NSET; ++s)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[s][r] = 0.f;
    // One step ahead, with one copy of the loading code: these launches are short enough to be bound by
    // instruction fetch (two unrolled buffers, 19-30 KB of code, took 12 us where this takes 5).
    float ca[16], cb[NSET][16];
    int cleft = 0;
#pragma unroll 1
    for (int t = t0; t <= t1; ++t) {
        float na[16], nb[NSET][16];
        int nleft = 0;
        if (t < t1) {
            const int src = t >= per_src ? 1 : 0;
            const long k0 = (long)(kb + t - src * per_src) * TK;
            nleft = p.K - k0 < TK ? (int)(p.K - k0) : TK;
            load_frag(na, p.A[src] + offA + k0 * p.sAk, p.sAk, nleft - 4 * lh, rowsA);
#pragma unroll
            for (int s = 0; s < NSET; ++s)
                load_frag(nb[s], p.B[NSET == 2 ? s : src] + offB + k0 * p.sBk, p.sBk, nleft - 4 * lh, rowsB);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (8 * j < cleft) {   // short contractions (few experts or segments) skip the zero padding
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int s = 0; s < NSET; ++s)
                        acc[s] = __builtin_amdgcn_mfma_f32_32x32x2f32(ca[4 * j + e], cb[s][4 * j + e], acc[s], 0, 0, 0);
            }
        }
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            ca[q] = na[q];
#pragma unroll
            for (int s = 0; s < NSET; ++s) cb[s][q] = nb[s][q];
        }
        cleft = nleft;
    }
    if (p.split_waves) {
        if (wave > 0) {
#pragma unroll
            for (int s = 0; s < NSET; ++s)
#pragma unroll
                for (int r = 0; r < 16; ++r) red[wave - 1][s][r][lane] = acc[s][r];
        }
        __syncthreads();
        if (wave > 0) return;
#pragma unroll
        for (int s = 0; s < NSET; ++s)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                acc[s][r] = ((acc[s][r] + red[0][s][r][lane]) + red[1][s][r][lane]) + red[2][s][r][lane];
    }

    // accumulator element r: row 8 (r >> 2) + 4 (lane >> 5) + (r & 3), column lane & 31
    const long n = n0 + l31;
    if (n >= p.N) return;
    const long rows = p.M - m0 - 4 * lh;   // rows left from the lane's first
    const size_t base = (size_t)(b * p.c_batch + (m0 + 4 * lh) * p.ldc + n);
    auto at = [&](int r) { return base + (size_t)((8 * (r >> 2) + (r & 3)) * p.ldc); };
    auto ok = [&](int r) { return 8 * (r >> 2) + (r & 3) < rows; };
    float x[16], y[16];   // what the epilogue reads, fetched together
    if constexpr (MODE == kGradAct) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (ok(r)) {
                x[r] = ew.G_in[at(r)];
                y[r] = ew.U_in[at(r)];
            }
    }
    float *C = p.C + (size_t)sl * p.c_slice;
    if (MODE == kStore && p.add) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (ok(r)) x[r] = C[at(r)];
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[0][r] += x[r];
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        if (!ok(r)) continue;
        const size_t o = at(r);
        const float v = acc[0][r];
        if constexpr (MODE == kStore) {
            C[o] = v;
        } else if constexpr (MODE == kGateUp) {
            const float u = acc[1][r];
            C[o] = v;
            ew.U[o] = u;
            if (ew.A) ew.A[o] = v * sigmoidf_(v) * u;
        } else {
            // v = dA:  dG = dA U sig(G) (1 + G (1 - sig(G))),  dU = dA G sig(G); also A (needed for dWd_bar)
            const float g = x[r], u = y[r], sg = sigmoidf_(g);
            ew.A[o] = g * sg * u;
            C[o] = v * u * sg * (1.0f + g * (1.0f - sg));
            ew.dU[o] = v * g * sg;
        }
    }
}

// ---------------------------------------------------------------- host helpers

struct F32Plan {
    int Sc;           // segments per chunk
    size_t slab;      // floats of one merged (or gradient) slab: Sc * D
    size_t act;       // floats of one activation buffer: Sc * T * d_ff
};

F32Plan plan(const Dims &m)
{
    const size_t per_seg = (size_t)4 * (6 * (size_t)m.D + 6 * (size_t)m.T * m.dff);
    long sc = (long)(kF32ChunkBudget / per_seg);
    if (sc < 1) sc = 1;
    if (sc > m.S) sc = m.S;
    F32Plan p;
    p.Sc = (int)sc;
    p.slab = (size_t)p.Sc * m.D;
    p.act = (size_t)p.Sc * m.T * m.dff;
    return p;
}

bool aligned(const float *q, long a, long b) { return ((uintptr_t)q & 15) == 0 && a % 4 == 0 && b % 4 == 0; }

// Operand strides: a row-major matrix with `ld` elements between rows; trans: the contraction runs along
// its rows' index (the stored matrix is [K][M] for A, [K][N] is the plain B).
Problem problem(int batches, long M, long N, long K, const float *A, long lda, long a_batch, bool ta, const float *B,
                long ldb, long b_batch, bool tb, float *C, long ldc, long c_batch)
{
    Problem p = {};
    p.A[0] = A; p.a_batch = a_batch;
    p.sAm = ta ? 1 : lda; p.sAk = ta ? lda : 1;
    p.B[0] = B; p.b_batch = b_batch;
    p.sBn = tb ? ldb : 1; p.sBk = tb ? 1 : ldb;
    p.C = C; p.ldc = ldc; p.c_batch = c_batch;
    p.M = M; p.N = N; p.K = K; p.batches = batches; p.ksplit = 1;
    p.vecA = aligned(A, lda, a_batch);
    p.vecB = aligned(B, ldb, b_batch);
    return p;
}

void second_source(Problem &p, const float *A, const float *B)
{
    p.A[1] = A; p.B[1] = B;
    p.vecA = p.vecA && aligned(A, 0, 0);
    p.vecB = p.vecB && aligned(B, 0, 0);
}

template <int MODE>
void launch(hipStream_t st, Group &g, const Elementwise &ew = Elementwise())
{
    long blocks = 0;
    for (int i = 0; i < g.n; ++i) {
        Problem &p = g.p[i];
        const long big = ((p.N + 63) / 64) * ((p.M + 63) / 64) * p.ksplit * p.batches;
        const long small = ((p.N + 31) / 32) * ((p.M + 31) / 32) * p.ksplit * p.batches;
        // Fewer than two tiles per CU: split the steps of a block over the wavefronts instead (down projection of 8 segments
        // of 128 tokens, d_ff = 256: 18.6 -> 6.6 us); a contraction of one step has nothing to split.
        p.split_waves = big < 512 && p.K > TK;
        p.blocks = (int)(p.split_waves ? small : big);
        blocks += p.blocks;
    }
    // A grid dimension counts fewer than 2^32 threads, i.e. 2^24 workgroups, which the expert gradients of
    // d * d_ff = 3.6e8 pass: further launches take the rest.  (2^31 workgroups of 64 x 64 elements would not fit
    // the memory.)
    for (long first = 0; first < blocks; first += kMaxGrid) {
        g.first = (int)first;
        const long n = blocks - first < kMaxGrid ? blocks - first : kMaxGrid;
        hipLaunchKernelGGL(contract_kernel<MODE>, dim3((unsigned)n), dim3(256), 0, st, g, ew);
    }
}

struct MergeArgs {
    const float *stack[3];
    float *slab[3];
};

// Merge of up to SB segments (grid y: blocks of segments, z: matrices): a thread owns VEC consecutive elements, keeps
// the sums of all SB segments and reads every expert once; the routing weights are uniform.  HBM-bound: one sequence, 4
// experts of 1024 x 2816 take 26 us (6.8 TB/s), 16 experts 112.  The contraction kernel, a workgroup of one step per 64
// columns, is bound by the rate at which workgroups start: 398 and 431.
template <int SB, int VEC>
__global__ __launch_bounds__(256) void merge_f32_kernel(const float *__restrict__ w, const MergeArgs m, int S, int E, long n)
{
    const long i = ((long)blockIdx.x * 256 + threadIdx.x) * VEC;
    if (i >= n) return;
    const int s0 = blockIdx.y * SB;
    const float *src = m.stack[blockIdx.z] + i;
    float acc[SB][VEC];
#pragma unroll
    for (int s = 0; s < SB; ++s)
#pragma unroll
        for (int j = 0; j < VEC; ++j) acc[s][j] = 0.f;
#pragma unroll 4
    for (int e = 0; e < E; ++e) {
        float v[VEC];
        if constexpr (VEC == 4) {
            const float4 f = *reinterpret_cast<const float4 *>(src + (size_t)e * n);
            v[0] = f.x; v[1] = f.y; v[2] = f.z; v[3] = f.w;
        } else {
            v[0] = src[(size_t)e * n];
        }
#pragma unroll
        for (int s = 0; s < SB; ++s) {
            const float ws = w[(size_t)(s0 + s < S ? s0 + s : S - 1) * E + e];
#pragma unroll
            for (int j = 0; j < VEC; ++j) acc[s][j] = fmaf(ws, v[j], acc[s][j]);
        }
    }
    float *dst = m.slab[blockIdx.z] + (size_t)s0 * n + i;
#pragma unroll
    for (int s = 0; s < SB; ++s) {
        if (s0 + s >= S) continue;
        if constexpr (VEC == 4)
            *reinterpret_cast<float4 *>(dst + (size_t)s * n) = make_float4(acc[s][0], acc[s][1], acc[s][2], acc[s][3]);
        else
            dst[(size_t)s * n] = acc[s][0];
    }
}

template <int SB>
void launch_merge(hipStream_t st, const float *w, int E, int S, long n, const MergeArgs &m, int count)
{
    bool vec = n % 4 == 0;
    for (int x = 0; x < count; ++x) vec = vec && aligned(m.stack[x], 0, 0) && aligned(m.slab[x], 0, 0);
    const long per = vec ? 4 : 1;
    const dim3 grid((unsigned)((n + 256 * per - 1) / (256 * per)), (S + SB - 1) / SB, count);
    if (vec)
        hipLaunchKernelGGL((merge_f32_kernel<SB, 4>), grid, dim3(256), 0, st, w, m, S, E, n);
    else
        hipLaunchKernelGGL((merge_f32_kernel<SB, 1>), grid, dim3(256), 0, st, w, m, S, E, n);
}

// slab_x[s][i] = sum_e w[s][e] stack_x[e][i]  for the given matrices
void merge(hipStream_t st, const float *w, int E, int Sc, long n, const float *const *stacks, float *const *slabs,
           int count)
{
    // Many experts for many segments are a contraction: blocks of 16 segments would read the stack again and again (us,
    // contraction / vectors: 64 segments, 40 experts, 1024 x 2816 1125 / 1457; 32 of 64 x 256 11.8 / 14.8).  Up to 16
    // experts or 8 segments the vectors win at every size tried (128 segments, 16 experts, 256 x 640 85 / 59; 8 and 40
    // 41 / 15), but for 10 % at 16 and 32 segments of the smallest matrices (50 x 130: 6.3 / 7.0).
    if (E <= 16 || Sc <= 8) {
        MergeArgs m = {};
        for (int x = 0; x < count; ++x) {
            m.stack[x] = stacks[x];
            m.slab[x] = slabs[x];
        }
        if (Sc == 1) return launch_merge<1>(st, w, E, Sc, n, m, count);
        if (Sc == 2) return launch_merge<2>(st, w, E, Sc, n, m, count);
        if (Sc <= 4) return launch_merge<4>(st, w, E, Sc, n, m, count);
        if (Sc <= 8) return launch_merge<8>(st, w, E, Sc, n, m, count);
        return launch_merge<16>(st, w, E, Sc, n, m, count);
    }
    Group g = {};
    g.n = count;
    for (int x = 0; x < count; ++x)
        g.p[x] = problem(1, Sc, n, E, w, E, 0, false, stacks[x], n, 0, false, slabs[x], n, 0);
    launch<kStore>(st, g);
}

void gate_up(hipStream_t st, const Dims &m, int sc, const float *X, const float *mg, const float *mu, float *G,
             float *U, float *A)
{
    const long TD = (long)m.T * m.d, TF = (long)m.T * m.dff;
    Group g = {};
    g.n = 1;
    g.p[0] = problem(sc, m.T, m.dff, m.d, X, m.d, TD, false, mg, m.dff, m.D, false, G, m.dff, TF);
    g.p[0].B[1] = mu;
    g.p[0].vecB = g.p[0].vecB && aligned(mu, 0, 0);
    Elementwise ew = {};
    ew.U = U;
    ew.A = A;
    launch<kGateUp>(st, g, ew);
}

}  // namespace

size_t f32_workspace_bytes(const Dims &m, int pass)
{
    const F32Plan p = plan(m);
    if (pass == LORY_PASS_FWD) return sizeof(float) * (3 * p.slab + 3 * p.act);
    return sizeof(float) * (6 * p.slab + 6 * p.act);
}

int f32_ffn_fwd(const Dims &m, const float *X, const float *w, const float *Wg, const float *Wu,
                const float *Wd, float *Y, float *G_save, float *U_save, void *ws, hipStream_t st)
{
    const F32Plan p = plan(m);
    float *mg = (float *)ws, *mu = mg + p.slab, *md = mu + p.slab;
    float *Gb = md + p.slab, *Ub = Gb + p.act, *Ab = Ub + p.act;
    const long TD = (long)m.T * m.d, TF = (long)m.T * m.dff;
    const float *stacks[3] = {Wg, Wu, Wd};
    float *slabs[3] = {mg, mu, md};
    for (int s0 = 0; s0 < m.S; s0 += p.Sc) {
        const int sc = (m.S - s0 < p.Sc) ? (m.S - s0) : p.Sc;
        merge(st, w + (size_t)s0 * m.E, m.E, sc, m.D, stacks, slabs, 3);
        gate_up(st, m, sc, X + (size_t)s0 * TD, mg, mu, G_save ? G_save + (size_t)s0 * TF : Gb,
                U_save ? U_save + (size_t)s0 * TF : Ub, Ab);
        Group g = {};
        g.n = 1;
        g.p[0] = problem(sc, m.T, m.d, m.dff, Ab, m.dff, TF, false, md, m.d, m.D, false, Y + (size_t)s0 * TD, m.d, TD);
        launch<kStore>(st, g);
    }
    return launch_status();
}

// Merged parameters of all m.S segments as [Wg_bar | Wu_bar | Wd_bar], each [S][rows][cols].
int f32_merge_all(const Dims &m, const float *w, const float *Wg, const float *Wu, const float *Wd,
                  float *Wbar, hipStream_t st)
{
    const float *stacks[3] = {Wg, Wu, Wd};
    float *slabs[3] = {Wbar, Wbar + (size_t)m.S * m.D, Wbar + (size_t)2 * m.S * m.D};
    merge(st, w, m.E, m.S, m.D, stacks, slabs, 3);
    return launch_status();
}

int f32_ffn_bwd(const Dims &m, const float *X, const float *w, const float *Wg, const float *Wu,
                const float *Wd, const float *dY, const float *G_save, const float *U_save,
                float *dX, float *dWg, float *dWu, float *dWd, int accumulate, float *dw, void *ws,
                hipStream_t st)
{
    const F32Plan p = plan(m);
    float *mg = (float *)ws, *mu = mg + p.slab, *md = mu + p.slab;
    float *gg = md + p.slab, *gu = gg + p.slab, *gd = gu + p.slab;
    float *Gb = gd + p.slab, *Ub = Gb + p.act, *Ab = Ub + p.act;
    float *parts = Ab + p.act, *dGb = parts + p.act, *dUb = dGb + p.act;
    const long TD = (long)m.T * m.d, TF = (long)m.T * m.dff;
    const float *stacks[3] = {Wg, Wu, Wd};
    float *slabs[3] = {mg, mu, md};
    const float *grads[3] = {gg, gu, gd};
    float *dW[3] = {dWg, dWu, dWd};
    for (int s0 = 0; s0 < m.S; s0 += p.Sc) {
        const int sc = (m.S - s0 < p.Sc) ? (m.S - s0) : p.Sc;
        const float *wc = w + (size_t)s0 * m.E;
        const float *Xc = X + (size_t)s0 * TD;
        const float *dYc = dY + (size_t)s0 * TD;
        merge(st, wc, m.E, sc, m.D, stacks, slabs, 3);
        const float *G = Gb, *U = Ub;
        if (G_save && U_save) {
            G = G_save + (size_t)s0 * TF;
            U = U_save + (size_t)s0 * TF;
        } else {
            gate_up(st, m, sc, Xc, mg, mu, Gb, Ub, nullptr);
        }
        // dA = dY Wd_bar^T, and from it dG, dU and A
        {
            Group g = {};
            g.n = 1;
            g.p[0] = problem(sc, m.T, m.dff, m.d, dYc, m.d, TD, false, md, m.d, m.D, true, dGb, m.dff, TF);
            Elementwise ew = {};
            ew.G_in = G; ew.U_in = U; ew.A = Ab; ew.dU = dUb;
            launch<kGradAct>(st, g, ew);
        }
        // dWg_bar = X^T dG ; dWu_bar = X^T dU ; dWd_bar = A^T dY
        {
            Group g = {};
            g.n = 3;
            g.p[0] = problem(sc, m.d, m.dff, m.T, Xc, m.d, TD, true, dGb, m.dff, TF, false, gg, m.dff, m.D);
            g.p[1] = problem(sc, m.d, m.dff, m.T, Xc, m.d, TD, true, dUb, m.dff, TF, false, gu, m.dff, m.D);
            g.p[2] = problem(sc, m.dff, m.d, m.T, Ab, m.dff, TF, true, dYc, m.d, TD, false, gd, m.d, m.D);
            launch<kStore>(st, g);
        }
        // dX = dG Wg_bar^T + dU Wu_bar^T; dWx[e] (+)= sum_s w[s,e] dWx_bar(s); partial sums of
        // <Wx[e], dWx_bar(s)> over slices of the matrix, 8 K steps or a little less each
        long slices = (m.D + 8 * TK - 1) / (8 * TK);
        const long room = (long)(p.act / ((size_t)3 * sc * m.E));
        if (slices > room) slices = room;
        if (slices > 128) slices = 128;
        const bool in_parts = slices >= 1;   // else (a few tokens) there is no room for partial sums
        {
            Group g = {};
            g.n = in_parts ? 7 : 4;
            g.p[0] = problem(sc, m.T, m.d, m.dff, dGb, m.dff, TF, false, mg, m.dff, m.D, true, dX + (size_t)s0 * TD, m.d, TD);
            second_source(g.p[0], dUb, mu);
            for (int x = 0; x < 3; ++x) {
                g.p[1 + x] = problem(1, m.E, m.D, sc, wc, m.E, 0, true, grads[x], m.D, 0, false, dW[x], m.D, 0);
                g.p[1 + x].add = (accumulate || s0 > 0) ? 1 : 0;
            }
            for (int x = 0; in_parts && x < 3; ++x) {
                Problem &q = g.p[4 + x];
                q = problem(1, sc, m.E, m.D, grads[x], m.D, 0, false, stacks[x], m.D, 0, true,
                            parts + (size_t)x * slices * sc * m.E, m.E, 0);
                q.ksplit = (int)slices;
                q.c_slice = (long)sc * m.E;
            }
            launch<kStore>(st, g);
            for (int x = 0; !in_parts && x < 3; ++x) {
                Group h = {};
                h.n = 1;
                h.p[0] = problem(1, sc, m.E, m.D, grads[x], m.D, 0, false, stacks[x], m.D, 0, true,
                                 dw + (size_t)s0 * m.E, m.E, 0);
                h.p[0].add = x > 0;
                launch<kStore>(st, h);
            }
        }
        if (in_parts) {
            if (k::launch_dw_reduce(st, parts, (int)(3 * slices), sc, m.E, dw + (size_t)s0 * m.E, sc, m.E) != hipSuccess)
                return LORY_ERR_DEVICE;
        }
    }
    return launch_status();
}

}  // namespace lory
