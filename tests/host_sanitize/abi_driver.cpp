// Walks the host-side layer of liblory (argument validation, shape checks, workspace and
// merged-save sizing with its block planning, the plans of the dense FFN, tuning knobs, the profiler's bookkeeping) for a
// build with -fsanitize=address,undefined on the host pass.  No call below reaches a kernel
// launch: every one returns from validation, or only computes sizes.
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include "lory.h"
#include "bf16_kernels.h"
#include "lory_internal.h"

static int failures = 0;
#define EXPECT(cond)                                                  \
    do {                                                              \
        if (!(cond)) {                                                \
            printf("FAILED line %d: %s\n", __LINE__, #cond);          \
            ++failures;                                               \
        }                                                             \
    } while (0)

static lory_shape shape(int B, int L, int T, int d, int dff, int E, int dtype)
{
    lory_shape s;
    s.B = B; s.L = L; s.T = T; s.d = d; s.d_ff = dff; s.E = E; s.dtype = dtype;
    return s;
}

int main()
{
    void *fake = (void *)(uintptr_t)0x7F0000001000ull;   // aligned, never dereferenced on these paths
    void *odd = (void *)(uintptr_t)0x7F0000001004ull;
    for (int i = -1; i < 9; ++i) EXPECT(lory_status_string(i) != NULL && strlen(lory_status_string(i)) > 0);
    EXPECT(strlen(lory_version()) >= 3);

    const int shapes[][7] = {
        {2, 512, 128, 64, 256, 4, LORY_F32},      {8, 4096, 256, 1024, 2816, 8, LORY_BF16},
        {8, 4096, 256, 1024, 2816, 32, LORY_BF16}, {4, 4096, 256, 2048, 5632, 32, LORY_BF16},
        {4, 4096, 64, 2048, 5632, 16, LORY_BF16},  {4, 4096, 1024, 2048, 5632, 16, LORY_BF16},
        {5, 3840, 64, 64, 128, 64, LORY_BF16},     {3, 60, 20, 50, 70, 5, LORY_F32},
        {4, 4096, 256, 4096, 11008, 4, LORY_BF16}, {1, 65536 * 64, 64, 64, 64, 1, LORY_BF16},
    };
    const size_t budgets[] = {(size_t)64 << 10, (size_t)1 << 20, (size_t)128 << 20, (size_t)6144 << 20};
    for (size_t b = 0; b < sizeof(budgets) / sizeof(budgets[0]); ++b) {
        EXPECT(lory_set_slab_budget(budgets[b]) == LORY_OK);
        for (int fused = 0; fused <= 2; ++fused) {
            EXPECT(lory_set_fused_merge(fused) == LORY_OK);
            for (size_t i = 0; i < sizeof(shapes) / sizeof(shapes[0]); ++i) {
                const int *q = shapes[i];
                const lory_shape s = shape(q[0], q[1], q[2], q[3], q[4], q[5], q[6]);
                size_t f = 0, w = 0, m = 0;
                const int rf = lory_workspace_bytes(&s, LORY_PASS_FWD, &f);
                const int rb = lory_workspace_bytes(&s, LORY_PASS_BWD, &w);
                const int rm = lory_merged_save_bytes(&s, &m);
                EXPECT(rf == rb && rb == rm);
                if (rf == LORY_OK) EXPECT(f > 0 && w >= f / 2 && f % 256 == 0 && w % 256 == 0);
            }
        }
    }
    EXPECT(lory_set_slab_budget(1024) == LORY_ERR_SHAPE);
    EXPECT(lory_set_fused_merge(4) == LORY_ERR_SHAPE && lory_set_fused_merge(-1) == LORY_ERR_SHAPE);
    EXPECT(lory_set_slab_budget((size_t)6144 << 20) == LORY_OK && lory_set_fused_merge(1) == LORY_OK);

    size_t out = 0;
    lory_shape ok = shape(2, 512, 128, 64, 256, 4, LORY_F32);
    lory_shape ragged = shape(2, 500, 128, 64, 256, 4, LORY_F32);
    lory_shape manyE = shape(2, 512, 128, 64, 256, 65, LORY_F32);
    lory_shape baddt = shape(2, 512, 128, 64, 256, 4, 7);
    lory_shape gran = shape(2, 512, 32, 64, 256, 4, LORY_BF16);
    EXPECT(lory_workspace_bytes(NULL, 0, &out) == LORY_ERR_NULL);
    EXPECT(lory_workspace_bytes(&ok, 0, NULL) == LORY_ERR_NULL);
    EXPECT(lory_workspace_bytes(&ok, 9, &out) == LORY_ERR_SHAPE);
    EXPECT(lory_workspace_bytes(&ragged, 0, &out) == LORY_ERR_SHAPE);
    EXPECT(lory_workspace_bytes(&manyE, 0, &out) == LORY_ERR_SHAPE);
    EXPECT(lory_workspace_bytes(&baddt, 0, &out) == LORY_ERR_DTYPE);
    EXPECT(lory_workspace_bytes(&gran, 0, &out) == LORY_ERR_SHAPE);
    lory_shape dense = shape(4, 1, 1, 2048, 5632, 1, LORY_BF16);
    EXPECT(lory_workspace_bytes(&dense, LORY_PASS_DENSE, &out) == LORY_OK && out > 0);

    // entry points: NULL, misaligned, small workspace -> status before any launch
    EXPECT(lory_route(&ok, NULL, fake, (float *)fake, NULL, NULL) == LORY_ERR_NULL);
    EXPECT(lory_route(&ok, odd, fake, (float *)fake, NULL, NULL) == LORY_ERR_ALIGN);
    EXPECT(lory_route(&ragged, fake, fake, (float *)fake, NULL, NULL) == LORY_ERR_SHAPE);
    EXPECT(lory_route_bwd(&ok, fake, (float *)fake, (float *)fake, (float *)fake, fake, NULL, 0, NULL) == LORY_ERR_NULL);
    EXPECT(lory_route_bwd(&ok, fake, (float *)fake, (float *)fake, (float *)fake, fake, (float *)fake, 2, NULL) ==
           LORY_ERR_SHAPE);
    EXPECT(lory_merged_ffn_fwd(&ok, fake, (float *)fake, fake, fake, fake, fake, NULL, NULL, NULL, fake, 16, NULL) ==
           LORY_ERR_WORKSPACE);
    EXPECT(lory_merged_ffn_fwd(&ok, fake, (float *)fake, fake, fake, fake, fake, fake, NULL, NULL, fake, 1 << 30,
                               NULL) == LORY_ERR_NULL);   // G without U
    EXPECT(lory_merged_ffn_fwd(&ok, fake, (float *)fake, fake, fake, fake, fake, NULL, NULL, fake, fake, 1 << 30,
                               NULL) == LORY_ERR_SHAPE);  // Wbar_save for fp32
    EXPECT(lory_merged_ffn_bwd(&ok, fake, (float *)fake, fake, fake, fake, fake, NULL, NULL, NULL, fake, fake, fake,
                               fake, LORY_BF16, 0, (float *)fake, fake, 1 << 30, NULL) == LORY_ERR_DTYPE);
    EXPECT(lory_merged_ffn_bwd(&ok, fake, (float *)fake, fake, fake, fake, fake, NULL, NULL, NULL, fake, fake, fake,
                               fake, LORY_F32, 3, (float *)fake, fake, 1 << 30, NULL) == LORY_ERR_SHAPE);
    EXPECT(lory_merged_ffn_bwd(&ok, fake, (float *)fake, fake, fake, fake, fake, NULL, NULL, NULL, fake, fake, fake,
                               fake, LORY_F32, 0, (float *)fake, fake, 16, NULL) == LORY_ERR_WORKSPACE);
    lory_shape inf = shape(2, 40, 40, 64, 128, 4, LORY_F32);
    lory_shape inf_bad = shape(2, 40, 20, 64, 128, 4, LORY_F32);
    EXPECT(lory_prompt_merge(&inf_bad, fake, NULL, fake, fake, fake, fake, (float *)fake, fake, NULL) == LORY_ERR_SHAPE);
    EXPECT(lory_prompt_merge(&inf, fake, NULL, fake, fake, fake, NULL, (float *)fake, fake, NULL) == LORY_ERR_NULL);
    EXPECT(lory_prompt_merge(&inf, fake, (const int32_t *)((char *)fake + 2), fake, fake, fake, fake, (float *)fake,
                             fake, NULL) == LORY_ERR_ALIGN);
    EXPECT(lory_dense_ffn_fwd(&inf, fake, fake, fake, fake, 16, NULL) == LORY_ERR_WORKSPACE);
    EXPECT(lory_dense_ffn_fwd_static(&inf, fake, NULL, fake, NULL) == LORY_ERR_NULL);
    lory_shape big = shape(2, 8, 8, 2048, 5632, 1, LORY_BF16);
    EXPECT(lory_dense_ffn_fwd_static(&big, fake, fake, fake, NULL) == LORY_ERR_WORKSPACE);

    // how the dense blocks of the GPU tests run (256 CUs): rows of a block, terms of the activation, tile height and
    // K slices of gate/up and down on the ring GEMM, K slices of down's last round of tiles, K slices of the projections
    // that stream their weights; every form that the dispatch has is among them
    static const struct { int B, L, d, dff; lory::DenseForm f; } forms[] = {
        // the ring GEMM
        {1, 65, 1664, 2816, {65, 2, 128, 11, 64, 8, 0, {0, 0}}},
        {2, 100, 512, 1408, {100, 2, 64, 0, 64, 9, 0, {0, 0}}},
        {3, 200, 64, 64, {200, 2, 64, 0, 64, 0, 0, {0, 0}}},
        {130, 100, 64, 64, {100, 2, 128, 0, 128, 0, 0, {0, 0}}},
        {150, 129, 64, 128, {129, 2, 192, 0, 192, 0, 0, {0, 0}}},
        {130, 250, 64, 64, {250, 2, 256, 0, 256, 0, 0, {0, 0}}},
        {40, 63, 192, 1728, {63, 2, 64, 0, 128, 6, 0, {0, 0}}},
        {16, 130, 320, 1408, {130, 2, 192, 0, 128, 2, 0, {0, 0}}},
        {40, 128, 192, 1728, {128, 1, 128, 0, 128, 6, 0, {0, 0}}},
        {1, 128, 320, 832, {128, 1, 64, 0, 64, 6, 0, {0, 0}}},
        {40, 65, 192, 1728, {65, 2, 128, 0, 64, 2, 0, {0, 0}}},
        {1, 50000, 64, 192, {16704, 2, 192, 0, 128, 0, 0, {0, 0}}},
        {4, 2001, 256, 704, {1024, 2, 128, 0, 64, 0, 0, {0, 0}}},
        {2, 17, 320, 832, {17, 2, 64, 0, 64, 6, 0, {0, 0}}},
        {4, 14, 1024, 4160, {14, 2, 64, 0, 64, 13, 0, {0, 0}}},
        {130, 11, 64, 704, {11, 2, 64, 0, 64, 3, 0, {0, 0}}},
        {6, 40, 1024, 1408, {40, 2, 64, 3, 128, 9, 0, {0, 0}}},
        // a last round of tiles that is cut
        {2, 2048, 768, 4160, {2048, 1, 192, 0, 256, 0, 5, {0, 0}}},
        {65, 128, 1024, 1024, {128, 1, 128, 0, 128, 0, 7, {0, 0}}},
        {65, 192, 1024, 1024, {192, 1, 192, 0, 192, 0, 7, {0, 0}}},
        {65, 256, 1024, 1024, {256, 1, 256, 0, 256, 0, 7, {0, 0}}},
        {66, 100, 1024, 1408, {100, 2, 128, 0, 128, 0, 9, {0, 0}}},
        {66, 180, 1024, 1024, {180, 2, 192, 0, 192, 0, 6, {0, 0}}},
        // contractions too long for the arithmetic of a slice stay whole
        {1, 64, 64, (1 << 24) + 64, {64, 1, 64, 0, 64, 0, 0, {0, 0}}},
        {1, 40, 64, (1 << 24) + 64, {40, 2, 64, 0, 64, 0, 0, {0, 0}}},
        // weights streamed: both projections
        {1, 1, 320, 832, {1, 2, 0, 0, 0, 0, 0, {4, 24}}},
        {5, 7, 320, 832, {7, 2, 0, 0, 0, 0, 0, {3, 4}}},
        {2, 1, 1088, 2880, {1, 2, 0, 0, 0, 0, 0, {2, 12}}},
        {1, 16, 64, 64, {16, 2, 0, 0, 0, 0, 0, {2, 1}}},
        {2, 16, 64, 1088, {16, 2, 0, 0, 0, 0, 0, {2, 12}}},
        {3, 9, 1088, 192, {9, 2, 0, 0, 0, 0, 0, {8, 1}}},
        {1, 2, 2560, 6144, {2, 2, 0, 0, 0, 0, 0, {2, 12}}},
        {17, 16, 128, 320, {16, 2, 0, 0, 0, 0, 0, {2, 3}}},
        {1, 16, 64, 12352, {16, 2, 0, 0, 0, 0, 0, {1, 32}}},
        {300, 1, 64, 192, {1, 2, 0, 0, 0, 0, 0, {1, 1}}},
        {1, 3, 64, 320, {3, 2, 0, 0, 0, 0, 0, {2, 1}}},
        {40, 2, 64, 448, {2, 2, 0, 0, 0, 0, 0, {1, 1}}},
        // gate/up alone
        {1, 17, 1024, 1088, {17, 2, 0, 0, 64, 7, 0, {4, 0}}},
        {1, 32, 1024, 1408, {32, 2, 0, 0, 64, 11, 0, {4, 0}}},
        {2, 33, 704, 832, {33, 2, 0, 0, 64, 6, 0, {3, 0}}},
        {3, 48, 1344, 320, {48, 2, 0, 0, 64, 2, 0, {6, 0}}},
        {1, 49, 2048, 128, {49, 2, 0, 0, 64, 0, 0, {16, 0}}},
        {2, 63, 1024, 832, {63, 2, 0, 0, 128, 6, 0, {4, 0}}},
        {1, 24, 2560, 64, {24, 2, 0, 0, 64, 0, 0, {16, 0}}},
    };
    for (size_t i = 0; i < sizeof(forms) / sizeof(forms[0]); ++i) {
        const lory_shape s = shape(forms[i].B, forms[i].L, forms[i].L, forms[i].d, forms[i].dff, 1, LORY_BF16);
        EXPECT(lory_workspace_bytes(&s, LORY_PASS_DENSE, &out) == LORY_OK);
        const lory::DenseForm f = lory::dense_form(lory::make_dims(s), out);
        if (memcmp(&f, &forms[i].f, sizeof(f)) != 0)
            printf("{%d, %d, %d, %d, {%d, %d, %d, %d, %d, %d, %d, {%d, %d}}},\n", s.B, s.L, s.d, s.d_ff, f.rows, f.terms, f.gu_tile,
                   f.gu_slices, f.down_tile, f.down_slices, f.down_pieces, f.stream.gu, f.stream.down);
        EXPECT(memcmp(&f, &forms[i].f, sizeof(f)) == 0);
    }
    // the same for the token GEMMs of the training steps in test_bf16_ring_gemm_cut_last_round: down, dA and dX
    static const struct { int B, L, T, d, dff, E; lory::LayerForm f; } layers[] = {
        {2, 960, 320, 320, 4160, 3, {{64, 4, 0}, {192, 0, 0}, {64, 4, 0}}},
        {3, 256, 64, 128, 4096, 17, {{64, 12, 0}, {64, 0, 0}, {64, 16, 0}}},
        {1, 2688, 192, 320, 4032, 3, {{64, 3, 0}, {192, 0, 0}, {192, 9, 0}}},
        {2, 1024, 256, 2880, 192, 3, {{128, 0, 0}, {64, 6, 0}, {128, 0, 0}}},
        {1, 4160, 64, 1024, 1536, 17, {{64, 10, 1}, {64, 0, 1}, {64, 16, 1}}},
        {5, 1664, 128, 1024, 384, 3, {{128, 0, 1}, {128, 0, 0}, {128, 6, 1}}},
        {5, 2496, 192, 1024, 384, 3, {{192, 0, 1}, {192, 0, 0}, {192, 6, 1}}},
    };
    for (size_t i = 0; i < sizeof(layers) / sizeof(layers[0]); ++i) {
        const lory_shape s = shape(layers[i].B, layers[i].L, layers[i].T, layers[i].d, layers[i].dff, layers[i].E, LORY_BF16);
        const lory::LayerForm f = lory::bf16_layer_form(lory::make_dims(s));
        if (memcmp(&f, &layers[i].f, sizeof(f)) != 0)
            printf("{%d, %d, %d, %d, %d, %d, {{%d, %d, %d}, {%d, %d, %d}, {%d, %d, %d}}},\n", s.B, s.L, s.T, s.d, s.d_ff, s.E,
                   f.down.rows, f.down.pieces, f.down.rounds, f.da.rows, f.da.pieces, f.da.rounds, f.dx.rows, f.dx.pieces,
                   f.dx.rounds);
        EXPECT(memcmp(&f, &layers[i].f, sizeof(f)) == 0);
    }
    // the reported workspace is what the planned form needs, and a larger one changes nothing
    unsigned rng = 12345;
    auto rnd = [&](int n) { rng = rng * 1664525u + 1013904223u; return (int)((rng >> 8) % (unsigned)n); };
    for (int i = 0; i < 20000; ++i) {
        lory_shape s = shape(1 + rnd(12), 1 + rnd(2048), 0, 64 * (1 + rnd(40)), 64 * (1 + rnd(96)), 1, LORY_BF16);
        s.T = s.L;
        EXPECT(lory_workspace_bytes(&s, LORY_PASS_DENSE, &out) == LORY_OK);
        const lory::DenseForm f = lory::dense_form(lory::make_dims(s), out);
        const lory::DenseForm g = lory::dense_form(lory::make_dims(s), (size_t)1 << 40);
        if (memcmp(&f, &g, sizeof(f)) != 0)
            printf("form %d x %d, %d, %d: down %d / %d, with more scratch %d / %d\n", s.B, s.L, s.d, s.d_ff, f.down_tile,
                   f.down_pieces, g.down_tile, g.down_pieces);
        EXPECT(memcmp(&f, &g, sizeof(f)) == 0);
    }

    // rounds of workgroups of a merge: a few prompts take one whatever the size, and one more sequence, expert or 64
    // columns changes the rounds by one step at most
    for (int d = 768; d <= 2560; d += 256)
        for (int f = 704; f <= 6144; f += 64)
            for (int e = 4; e <= 64; ++e)
                for (int s = 1; s <= 12; ++s) EXPECT(lory::k::merge_rounds(e, s, (long)d * f, false) == 1 || s > 10 + e / 4);
    for (int t = 0; t < 2; ++t)
        for (int f = 704; f <= 6144; f += 64)
            for (int e = 4; e <= 32; ++e)
                for (int s = 1; s <= 128; ++s) {
                    const int r = lory::k::merge_rounds(e, s, 2048L * f, t);
                    const int n[3] = {lory::k::merge_rounds(e, s + 1, 2048L * f, t), lory::k::merge_rounds(e + 1, s, 2048L * f, t),
                                      lory::k::merge_rounds(e, s, 2048L * (f + 64), t)};
                    for (int i = 0; i < 3; ++i) EXPECT(n[i] <= 2 * r && r <= 2 * n[i]);
                }

    // profiler bookkeeping without launches
    lory_kernel_stat st[8];
    int n = -1;
    EXPECT(lory_profile_read(NULL, 8, &n) == LORY_ERR_NULL);
    EXPECT(lory_profile_read(st, 0, &n) == LORY_ERR_SHAPE);
    EXPECT(lory_profile_read(st, 8, &n) == LORY_OK && n == 0);

    printf("abi sanitizer run: %s (%d failures)\n", failures ? "FAILED" : "ok", failures);
    return failures ? 1 : 0;
}
