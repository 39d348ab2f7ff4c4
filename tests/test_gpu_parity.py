"""GPU parity: the HIP library (through the C ABI) against the CPU fp64
oracle, element by element on the same seeded inputs.

Tolerances (relative L2 per output tensor): 1e-5 for the fp32 configuration,
1e-2 for bf16 operands with fp32 accumulation.
"""
import ctypes

import numpy as np
import pytest
import torch

from oracle import lory_oracle as orc
from paper_2405_03133_amd import binding as lb
from paper_2405_03133_amd.inputs import CONFIGS, LoryConfig, make_inputs, make_routing_weights, round_to_bf16
from parity_util import check, host, rel_l2

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 1e-2}
# Router-weight gradient of the whole layer: dR = sum_s hbar_s^T dz_s, dz = e * (de - <e, de>), de = the
# FFN's dw shifted by one segment.  It inherits the error of dw (the bar above; the centring
# de - <e, de> is well conditioned for these inputs, ||de|| / ||de - <e, de>|| is about 1) and of the
# fp32 softmax and segment means of the forward (1e-7 relative), hence 1e-4 instead of 1e-5 for the
# fp32 configuration, as for lory_route_bwd on its own.
DR_TOL = {"f32": 1e-4, "bf16": 1e-2}


def tdtype(cfg):
    return torch.float32 if cfg.dtype == "f32" else torch.bfloat16


def to_dev(a, cfg):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda().to(tdtype(cfg)).contiguous()


def run_layer(cfg, t, w_override=None, save=True, grad_dtype=torch.float32, merged_save=False):
    """route -> fwd -> bwd on the GPU through the C ABI; returns numpy float64."""
    print(f"[gpu] {cfg}", flush=True)
    X, R = to_dev(t["X"], cfg), to_dev(t["R"], cfg)
    Wg, Wu, Wd = (to_dev(t[k], cfg) for k in ("Wg", "Wu", "Wd"))
    dY = to_dev(t["dY"], cfg)
    hbar = torch.empty((cfg.S, cfg.d), dtype=torch.float32, device="cuda")
    w = lb.lory_route(X, R, cfg.T, hbar=hbar, d_ff=cfg.d_ff)
    w_used = w if w_override is None else torch.from_numpy(w_override).cuda().float().contiguous()
    G = U = None
    if save:
        G = torch.empty((cfg.tokens, cfg.d_ff), dtype=X.dtype, device="cuda")
        U = torch.empty_like(G)
    Wbar = None
    if merged_save:
        Wbar = lb.alloc_merged_save(lb.make_shape(cfg.B, cfg.L, cfg.T, cfg.d, cfg.d_ff, cfg.E, X.dtype))
        assert Wbar is not None
    Y = lb.lory_merged_ffn_fwd(X, w_used, Wg, Wu, Wd, cfg.T, G_save=G, U_save=U, Wbar_save=Wbar)
    dX, dWg, dWu, dWd, dw = lb.lory_merged_ffn_bwd(X, w_used, Wg, Wu, Wd, dY, cfg.T, G_save=G, U_save=U,
                                                   grad_dtype=grad_dtype, Wbar_save=Wbar)
    torch.cuda.synchronize()
    out = {"w": host(w), "hbar": host(hbar), "Y": host(Y), "dX": host(dX), "dWg": host(dWg),
           "dWu": host(dWu), "dWd": host(dWd), "dw": host(dw), "w_used": host(w_used)}
    if save:
        out["G"], out["U"] = host(G), host(U)
    return out


def oracle_layer(cfg, t, w_used):
    r = orc.route(t["X"], t["R"], cfg.T)
    f = orc.ffn_fwd(t["X"], w_used, t["Wg"], t["Wu"], t["Wd"], cfg.T, want_gu=True)
    g = orc.ffn_bwd(t["X"], w_used, t["Wg"], t["Wu"], t["Wd"], t["dY"], cfg.T)
    out = {"w": r["w"], "hbar": r["hbar"], "Y": f["Y"], "G": f["G"], "U": f["U"]}
    out.update(g)
    return out


def compare(cfg, got, ref, names, tol):
    """Whole-tensor rel-L2, worst-row rel-L2 and largest absolute error of every named tensor
    (parity_util.check: the last two are what a single wrong tile or ragged last block trips)."""
    return {k: check(f"{cfg.name} {k}", got[k], ref[k], tol) for k in names}


ALL = ("Y", "G", "U", "dX", "dWg", "dWu", "dWd", "dw")


# ------------------------------------------------------------------ fp32

@pytest.mark.parametrize("structured", [False, True])
def test_c1_fp32_route_fwd_bwd(structured):
    cfg = CONFIGS["C1"]
    t = make_inputs(cfg, structured=structured)
    got = run_layer(cfg, t)
    # the FFN is checked with the GPU's own routing weights as the oracle's input,
    # the routing weights themselves against the oracle's route
    ref = oracle_layer(cfg, t, got["w_used"])
    compare(cfg, got, ref, ("w", "hbar"), 1e-6)
    np.testing.assert_allclose(got["w"].sum(-1), 1.0, atol=1e-6)
    compare(cfg, got, ref, ALL, TOL["f32"])


@pytest.mark.parametrize("cfg", [
    LoryConfig("f32_ragged_dims", B=3, L=60, T=20, d=50, d_ff=70, E=5, dtype="f32", seed=21),
    LoryConfig("f32_single_segment", B=2, L=48, T=48, d=32, d_ff=96, E=3, dtype="f32", seed=22),
    LoryConfig("f32_one_expert", B=1, L=64, T=16, d=24, d_ff=40, E=1, dtype="f32", seed=23),
    LoryConfig("f32_max_experts", B=1, L=32, T=8, d=16, d_ff=24, E=64, dtype="f32", seed=24),
    LoryConfig("f32_one_token_segments", B=2, L=6, T=1, d=12, d_ff=20, E=4, dtype="f32", seed=25),
], ids=lambda c: c.name)
def test_fp32_edge_shapes(cfg):
    t = make_inputs(cfg, structured=True)
    got = run_layer(cfg, t, save=(cfg.E != 1))
    ref = oracle_layer(cfg, t, got["w_used"])
    compare(cfg, got, ref, ("w", "hbar"), 1e-6)
    names = ALL if cfg.E != 1 else ("Y", "dX", "dWg", "dWu", "dWd", "dw")
    compare(cfg, got, ref, names, TOL["f32"])


# The contraction kernel where it can go wrong: no room for partial inner products (fewer activations than
# routing weights), more than one step over experts and segments with rows that are not 16-byte aligned, and
# enough tiles that the wavefronts of a workgroup work on blocks of their own.
@pytest.mark.parametrize("cfg", [
    LoryConfig("f32_no_room", B=3, L=4, T=1, d=8, d_ff=8, E=16, dtype="f32", seed=27),
    LoryConfig("f32_two_steps", B=4, L=400, T=40, d=72, d_ff=130, E=40, dtype="f32", seed=28),
    LoryConfig("f32_many_tiles", B=8, L=1024, T=128, d=96, d_ff=200, E=9, dtype="f32", seed=29),
], ids=lambda c: c.name)
@pytest.mark.parametrize("save", [True, False], ids=["saved_GU", "recompute_GU"])
def test_fp32_contraction_forms(cfg, save):
    t = make_inputs(cfg, structured=True)
    got = run_layer(cfg, t, save=save)
    names = ALL if save else ("Y", "dX", "dWg", "dWu", "dWd", "dw")
    compare(cfg, got, oracle_layer(cfg, t, got["w_used"]), names, TOL["f32"])


# Routing where its thread layout changes: expert counts around 16, 32 and 64 lanes per row of R; widths around the
# 64, 128 and 256 column threads (one column each when a row is not a multiple of a 16-byte load); segments of fewer,
# as many and more rows than the rounds of eight; the path that returns the means and the one that does not; and
# the mean of a whole prompt, whose last chunk of 64 rows is short.  The bound is the one of fp32 sums.
@pytest.mark.parametrize("dtype,d,T,E", [
    ("f32", 63, 5, 1), ("f32", 255, 33, 15), ("f32", 260, 40, 17), ("f32", 513, 70, 64), ("f32", 1028, 300, 33),
    ("bf16", 64, 64, 16), ("bf16", 512, 128, 32), ("bf16", 576, 192, 33), ("bf16", 1088, 320, 12),
    ("bf16", 2112, 64, 64),
])
def test_route_forms(dtype, d, T, E):
    cfg = LoryConfig("route", B=2, L=3 * T, T=T, d=d, d_ff=64, E=E, dtype=dtype, seed=31)
    t = make_inputs(cfg, structured=True, with_dy=False)
    X, R = to_dev(t["X"], cfg), to_dev(t["R"], cfg)
    hbar = torch.empty((cfg.S, d), dtype=torch.float32, device="cuda")
    print(f"[gpu] {cfg}", flush=True)
    w_h, w = lb.lory_route(X, R, T, hbar=hbar, d_ff=64), lb.lory_route(X, R, T, d_ff=64)
    w_p, _ = lb.lory_prompt_merge(X, R, *(to_dev(t[k], cfg) for k in ("Wg", "Wu", "Wd")))
    ref = orc.route(t["X"], t["R"], T)
    check("w, means returned", host(w_h), ref["w"], TOL["f32"])
    check("hbar", host(hbar), ref["hbar"], TOL["f32"])
    check("w", host(w), ref["w"], TOL["f32"])
    check("w, prompt", host(w_p), orc.route(t["X"], t["R"], cfg.L)["w"], TOL["f32"])


# fp32 merges: one to 16 segments per thread with a short last block, rows of matrices that are not 16-byte aligned, and
# the contraction for many experts and segments.  Sums of at most 40 products in fp32.
@pytest.mark.parametrize("B,E", [(1, 3), (2, 40), (3, 5), (8, 17), (9, 16), (9, 17), (17, 4), (33, 16), (40, 20)])
@pytest.mark.parametrize("d,d_ff", [(7, 9), (24, 10), (40, 36)])
def test_fp32_merge_forms(B, E, d, d_ff):
    gen = torch.Generator(device="cuda").manual_seed(B + E)
    X, R = torch.randn((B, 3, d), generator=gen, device="cuda"), torch.randn((d, E), generator=gen, device="cuda")
    W = [torch.randn(s, generator=gen, device="cuda") for s in ((E, d, d_ff), (E, d, d_ff), (E, d_ff, d))]
    w, Wbar = lb.lory_prompt_merge(X, R, *W, Wbar=torch.full((3, B, d * d_ff), float("nan"), device="cuda"))
    for i in range(3):
        ref = host(w) @ host(W[i]).reshape(E, -1)
        assert np.abs(host(Wbar[i]) - ref).max() <= 40 * 2.0 ** -24 * np.abs(host(W[i])).max(), i


def test_fp32_very_large_matrices():
    """Matrices whose workgroups exceed what one launch counts: the merge of one expert is a copy, and the expert
    gradients of one token are outer products."""
    d, d_ff = 16384, 21888
    gen = torch.Generator(device="cuda").manual_seed(5)
    X, dY = (torch.randn((1, 1, d), generator=gen, device="cuda") for _ in range(2))
    W = [torch.empty(s, device="cuda").uniform_(-0.01, 0.01, generator=gen) for s in ((1, d, d_ff), (1, d, d_ff), (1, d_ff, d))]
    print(f"[gpu] d={d} d_ff={d_ff}", flush=True)
    w, Wbar = lb.lory_prompt_merge(X, torch.ones((d, 1), device="cuda"), *W,
                                   Wbar=torch.full((3, 1, d * d_ff), float("nan"), device="cuda"))
    assert w.item() == 1.0
    for i in range(3):
        assert torch.equal(Wbar[i].view(-1), W[i].view(-1)), i
    del Wbar
    grads = [torch.full(t.shape, float("nan"), device="cuda") for t in W]
    dX = lb.lory_merged_ffn_bwd(X, w, *W, dY, 1, dWg=grads[0], dWu=grads[1], dWd=grads[2], grad_dtype=torch.float32)[0]
    x, dy = X[0, 0].double(), dY[0, 0].double()

    def mv(m, v):   # m @ v and m.T @ v without a copy of m in 64 bits
        return (torch.mv(m[0], v.float()) if m.shape[2] == v.numel() else torch.mv(m[0].t(), v.float())).double()

    g, u, da = mv(W[0], x), mv(W[1], x), mv(W[2], dy)
    sg = torch.sigmoid(g)
    dg, du, a = da * u * sg * (1 + g * (1 - sg)), da * g * sg, g * sg * u
    tol = 1e-4   # sums of 16384 .. 21888 products in fp32 on both sides
    for got, (col, row) in zip(grads, ((x, dg), (x, du), (a, dy))):
        err = sum(float((got[0, i:i + 1024].double() - col[i:i + 1024, None] * row).pow(2).sum())
                  for i in range(0, got.shape[1], 1024)) ** 0.5
        assert err <= tol * float(col.norm() * row.norm())
    ref = mv(W[0], dg) + mv(W[1], du)
    assert float((dX[0, 0].double() - ref).norm()) <= tol * float(ref.norm())


def test_fp32_given_routing_weights_onehot_and_accumulate():
    cfg = CONFIGS["C1"]
    t = make_inputs(cfg)
    w1 = make_routing_weights(cfg, "onehot")
    got = run_layer(cfg, t, w_override=w1)
    ref = oracle_layer(cfg, t, w1)
    compare(cfg, got, ref, ALL, TOL["f32"])
    # accumulate=1 adds to existing gradient stacks; dX and dw are overwritten
    X, Wg, Wu, Wd, dY = (to_dev(t[k], cfg) for k in ("X", "Wg", "Wu", "Wd", "dY"))
    w = torch.from_numpy(w1).cuda()
    base = [torch.full_like(Wg, 0.5), torch.full_like(Wu, -0.25), torch.full_like(Wd, 2.0)]
    dX, dWg, dWu, dWd, dw = lb.lory_merged_ffn_bwd(X, w, Wg, Wu, Wd, dY, cfg.T, dWg=base[0], dWu=base[1],
                                                   dWd=base[2], accumulate=True)
    torch.cuda.synchronize()
    assert rel_l2(host(dWg) - 0.5, ref["dWg"]) <= 1e-4
    assert rel_l2(host(dWu) + 0.25, ref["dWu"]) <= 1e-4
    assert rel_l2(host(dWd) - 2.0, ref["dWd"]) <= 1e-4
    assert rel_l2(host(dX), ref["dX"]) <= TOL["f32"]
    assert rel_l2(host(dw), ref["dw"]) <= TOL["f32"]


def test_errors_leave_outputs_untouched():
    cfg = CONFIGS["C1"]
    t = make_inputs(cfg)
    X, Wg, Wu, Wd = (to_dev(t[k], cfg) for k in ("X", "Wg", "Wu", "Wd"))
    w = torch.full((cfg.S, cfg.E), 1.0 / cfg.E, device="cuda")
    Y = torch.full_like(X, 7.0)
    tiny_ws = torch.empty(256, dtype=torch.uint8, device="cuda")
    with pytest.raises(lb.LoryError) as ei:
        lb.lory_merged_ffn_fwd(X, w, Wg, Wu, Wd, cfg.T, Y=Y, workspace=tiny_ws)
    assert ei.value.status == lb.LORY_ERR_WORKSPACE
    torch.cuda.synchronize()
    assert bool((Y == 7.0).all())
    # the library stays usable
    lb.lory_merged_ffn_fwd(X, w, Wg, Wu, Wd, cfg.T, Y=Y)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(Y).all()) and not bool((Y == 7.0).all())


# ------------------------------------------------------------------ bf16

BF16_CASES = [
    # (config, slab budget in bytes) - small budgets force several blocks and a ragged last block
    (LoryConfig("bf16_multi_block", B=2, L=512, T=128, d=256, d_ff=576, E=8, dtype="bf16", seed=31), 1 << 20),
    (LoryConfig("bf16_T64", B=2, L=256, T=64, d=128, d_ff=192, E=4, dtype="bf16", seed=32), 256 << 10),
    (LoryConfig("bf16_T256_E32", B=1, L=512, T=256, d=192, d_ff=256, E=32, dtype="bf16", seed=33), 512 << 10),
    (LoryConfig("bf16_E33", B=1, L=256, T=64, d=64, d_ff=128, E=33, dtype="bf16", seed=34), 128 << 20),
    (LoryConfig("bf16_S40", B=5, L=512, T=64, d=64, d_ff=64, E=3, dtype="bf16", seed=35), 128 << 20),
    (LoryConfig("bf16_one_expert", B=1, L=128, T=64, d=64, d_ff=128, E=1, dtype="bf16", seed=36), 128 << 20),
    # segment counts and lengths of the benchmark configurations at reduced widths
    (LoryConfig("bf16_S128_E32", B=8, L=4096, T=256, d=128, d_ff=256, E=32, dtype="bf16", seed=37), 4 << 20),
    (LoryConfig("bf16_S256_T64_E16", B=4, L=4096, T=64, d=128, d_ff=256, E=16, dtype="bf16", seed=38), 128 << 20),
    (LoryConfig("bf16_T1024_E16", B=1, L=2048, T=1024, d=128, d_ff=256, E=16, dtype="bf16", seed=39), 128 << 20),
    (LoryConfig("bf16_S300_E64", B=5, L=3840, T=64, d=64, d_ff=128, E=64, dtype="bf16", seed=40), 128 << 20),
    # 129-256 segments with at most 16 experts: the scatter instance that parks its expert chunks in LDS,
    # here with fewer 16-segment blocks than its static bound
    (LoryConfig("bf16_S160_E12", B=5, L=2048, T=64, d=64, d_ff=128, E=12, dtype="bf16", seed=44), 128 << 20),
    # every GEMM on the persistent ring kernel with two tiles per workgroup (tile boundaries inside
    # the K-step stream), all outputs compared element by element
    (LoryConfig("bf16_ring_two_tiles", B=4, L=4096, T=256, d=512, d_ff=1024, E=4, dtype="bf16", seed=43),
     6144 << 20),
]


@pytest.fixture
def default_budget():
    yield
    lb.lory_set_slab_budget(6144 << 20)


@pytest.mark.parametrize("cfg,budget", BF16_CASES, ids=lambda v: v.name if isinstance(v, LoryConfig) else str(v))
def test_bf16_small_shapes(cfg, budget, default_budget):
    lb.lory_set_slab_budget(budget)
    t = make_inputs(cfg, structured=True)
    got = run_layer(cfg, t)
    ref = oracle_layer(cfg, t, got["w_used"])
    compare(cfg, got, ref, ("w", "hbar"), 1e-5)
    compare(cfg, got, ref, ALL, TOL["bf16"])


# Shapes whose GEMMs need edge tiles of every height (T or d_ff no multiple of the tile) and several tiles
# per workgroup, so that edge tiles sit inside the stream of K steps.
RING_EDGE_CASES = [
    LoryConfig("ring_192_rows", B=4, L=4608, T=192, d=320, d_ff=832, E=3, dtype="bf16", seed=45),
    LoryConfig("ring_128_rows_clamped", B=2, L=3840, T=320, d=320, d_ff=832, E=3, dtype="bf16", seed=46),
    LoryConfig("ring_256_rows_clamped", B=2, L=4032, T=448, d=320, d_ff=832, E=3, dtype="bf16", seed=47),
    LoryConfig("ring_64_rows", B=2, L=1280, T=64, d=192, d_ff=704, E=20, dtype="bf16", seed=48),
    LoryConfig("ring_smallest", B=1, L=64, T=64, d=64, d_ff=64, E=2, dtype="bf16", seed=49),
]


@pytest.mark.parametrize("cfg", RING_EDGE_CASES, ids=lambda c: c.name)
def test_bf16_ring_gemm_edge_tiles(cfg):
    t = make_inputs(cfg, structured=True)
    got = run_layer(cfg, t)
    compare(cfg, got, oracle_layer(cfg, t, got["w_used"]), ALL, TOL["bf16"])


@pytest.mark.parametrize("cfg", RING_EDGE_CASES, ids=lambda c: c.name)
def test_bf16_ring_gemm_edge_tiles_without_saved_planes(cfg):
    """The gate/up instance that writes the activation alone."""
    t = make_inputs(cfg, structured=True, with_dy=False)
    print(f"[gpu] {cfg}", flush=True)
    w = orc.route(t["X"], t["R"], cfg.T)["w"].astype(np.float32)
    Y = lb.lory_merged_ffn_fwd(to_dev(t["X"], cfg), torch.from_numpy(w).cuda(), *(to_dev(t[k], cfg) for k in ("Wg", "Wu", "Wd")),
                               cfg.T)
    ref = orc.ffn_fwd(t["X"], w.astype(np.float64), t["Wg"], t["Wu"], t["Wd"], cfg.T)["Y"]
    check(f"{cfg.name} Y", host(Y), ref, TOL["bf16"])


# Segments with equal routing rows share their merged values: runs that start, end and cross at the 32- and 64-segment
# words, one run over everything, rows equal but not adjacent, and none.  The saved mode stores every segment, so its bits
# are the reference for the sharing mode's.
@pytest.mark.parametrize("cfg", [
    LoryConfig("shared_S150", B=5, L=3840, T=128, d=64, d_ff=128, E=5, dtype="bf16", seed=111),
    LoryConfig("shared_E33", B=2, L=4096, T=128, d=64, d_ff=64, E=33, dtype="bf16", seed=112),
    # few segments: merge_few_kernel, two units and one unit a wavefront
    LoryConfig("shared_S15", B=3, L=640, T=128, d=64, d_ff=192, E=5, dtype="bf16", seed=123),
    LoryConfig("shared_S8", B=2, L=512, T=128, d=64, d_ff=192, E=33, dtype="bf16", seed=124),
], ids=lambda c: c.name)
@pytest.mark.parametrize("runs", ["words", "all", "alternating", "none"])
def test_bf16_equal_routing_rows(cfg, runs):
    t = make_inputs(cfg, structured=True)
    w = make_routing_weights(cfg, "peaked")
    if runs == "words":
        for a, b in ((0, 2), (31, 33), (40, 64), (64, 66), (100, cfg.S)):
            w[a:min(b, cfg.S)] = w[a if a < cfg.S else 0]
    elif runs == "all":
        w[:] = w[0]
    elif runs == "alternating":
        w[0::2], w[1::2] = w[0], w[1]
    w = np.ascontiguousarray(w, dtype=np.float32)
    for save in (True, False):   # the second recomputes G and U in the backward
        got, saved = (run_layer(cfg, t, w_override=w, save=save, merged_save=m) for m in (False, True))
        for key in ("Y", "dX", "dWg", "dWu", "dWd", "dw"):
            assert np.array_equal(got[key], saved[key]), key


# Every form of the merge of few segments (up to 8 and 16 segments; up to 8 experts two units a wavefront, else one), with
# remainders of the experts; (9, 9) and (17, 3) are beyond the line and merged by merge_kernel.
@pytest.mark.parametrize("B,E,d,d_ff", [(1, 1, 64, 64), (1, 13, 64, 320), (2, 2, 128, 192), (3, 7, 64, 128), (4, 8, 192, 64),
                                        (5, 11, 64, 64), (6, 9, 64, 192), (7, 16, 64, 64), (8, 33, 64, 128), (11, 6, 64, 64),
                                        (12, 8, 64, 192), (14, 3, 64, 128), (16, 6, 64, 64), (9, 9, 64, 64), (13, 7, 64, 192),
                                        (17, 3, 64, 64)])
def test_bf16_merge_of_few_segments(B, E, d, d_ff):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000 * B + E)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda").bfloat16()
    X, R, W = rand(B, 64, d), rand(d, E), [rand(E, d, d_ff), rand(E, d, d_ff), rand(E, d_ff, d)]
    print(f"[gpu] few segments B={B} E={E}", flush=True)
    w, Wbar = lb.lory_prompt_merge(X, R, *W, Wbar=torch.full((3, B, d * d_ff), float("nan"), device="cuda", dtype=torch.bfloat16))
    w64 = host(w).astype(np.float64)
    for x in range(3):
        st = host(W[x]).astype(np.float64).reshape(E, -1)
        ref, mag = w64 @ st, np.abs(w64) @ np.abs(st)
        # one rounding to bf16, and sums in 32 bits of weights that the matrix cores take as hi + lo (2^-17)
        assert np.all(np.abs(host(Wbar[x]) - ref) <= 2.0 ** -8 * np.abs(ref) + 2.0 ** -15 * mag), x


# The merged parameters of a prompt have the same bits whatever number of prompts is merged beside it: every count of
# register sets and units (up to 8, 16, 32, 48 and 64 experts), on both sides of where merge_kernel takes over.
@pytest.mark.parametrize("E,counts", [(3, (1, 8, 9, 16, 17)), (8, (2, 12, 16, 33)), (9, (1, 5, 8, 9)), (16, (3, 8, 20)),
                                      (32, (1, 7, 8, 9)), (40, (2, 8, 9)), (64, (1, 4, 8, 9))])
def test_bf16_merged_prompt_does_not_depend_on_the_batch(E, counts):
    print(f"[gpu] merged prompts {E} {counts}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(130)
    d, d_ff, n = 64, 192, max(counts)
    X = (torch.randn((n, 40, d), generator=gen, device="cuda") + torch.randn((n, 1, d), generator=gen, device="cuda")).bfloat16()
    R = (torch.randn((d, E), generator=gen, device="cuda") / 8).bfloat16()
    Wg, Wu, Wd = (torch.randn(s, generator=gen, device="cuda").mul_(0.02).bfloat16() for s in ((E, d, d_ff), (E, d, d_ff), (E, d_ff, d)))
    w, Wbar = lb.lory_prompt_merge(X, R, Wg, Wu, Wd)
    for B in counts:
        wb, part = lb.lory_prompt_merge(X[:B].contiguous(), R, Wg, Wu, Wd)
        assert torch.equal(wb, w[:B]) and torch.equal(part, Wbar[:, :B]), B


def test_profile_counts_shared_merges_once():
    """Bytes of the merges and of the GEMMs behind them: merged values of segments with equal routing rows are
    written and read once; saved merged parameters are written for every segment."""
    cfg = LoryConfig("profile_shared", B=3, L=1280, T=128, d=128, d_ff=192, E=4, dtype="bf16", seed=114)
    t = make_inputs(cfg, structured=True)
    w = make_routing_weights(cfg, "peaked")
    w[7:12], w[29] = w[7], w[28]     # five segments of one row, and the last pair
    S, D, tok = cfg.S, cfg.d * cfg.d_ff, cfg.tokens
    kept = 1 + sum(not np.array_equal(w[s], w[s - 1]) for s in range(1, S))
    assert kept <= S - 5
    for merged_save, n in ((False, kept), (True, S)):
        lb.lory_profile_enable(True)
        try:
            lb.lory_profile_read()
            run_layer(cfg, t, w_override=w, merged_save=merged_save)
            stats = {s["name"]: s for s in lb.lory_profile_read()}
        finally:
            lb.lory_profile_enable(False)
        merges = 3 if merged_save else 6
        assert stats["merge"]["launches"] == merges
        assert stats["merge"]["bytes"] == 2.0 * D * (cfg.E + n) * merges
        acts = 2.0 * tok * (cfg.d + cfg.d_ff)
        assert stats["gemm_gate_up"]["bytes"] == acts + 2.0 * tok * cfg.d_ff + 4.0 * n * D   # G and U are saved
        assert stats["gemm_down"]["bytes"] == acts + 2.0 * n * D
        assert stats["gemm_dA"]["bytes"] == acts + 2.0 * n * D
        assert stats["gemm_dX"]["bytes"] == acts + 2.0 * tok * cfg.d_ff + 4.0 * n * D


def test_bf16_forward_in_place():
    """Y may be X: the down projection writes it after everything that reads X."""
    cfg = LoryConfig("in_place", B=2, L=512, T=128, d=128, d_ff=192, E=4, dtype="bf16", seed=113)
    t = make_inputs(cfg, structured=True, with_dy=False)
    X, Wg, Wu, Wd = (to_dev(t[k], cfg) for k in ("X", "Wg", "Wu", "Wd"))
    w = lb.lory_route(X, to_dev(t["R"], cfg), cfg.T, d_ff=cfg.d_ff)
    Y = lb.lory_merged_ffn_fwd(X, w, Wg, Wu, Wd, cfg.T)
    Z = X.clone()
    lb.lory_merged_ffn_fwd(Z, w, Wg, Wu, Wd, cfg.T, Y=Z)
    torch.cuda.synchronize()
    assert torch.equal(Y, Z)


# A last round of tiles cut over K: with and without whole rounds before it, edge tiles, K slices that begin in the first or
# second source of dX or span both, and slices of different lengths.  tests/host_sanitize/abi_driver.cpp pins the tile heights,
# the slices and the whole rounds of each contraction.
TAIL_CASES = [
    LoryConfig("tail_T320", B=2, L=960, T=320, d=320, d_ff=4160, E=3, dtype="bf16", seed=101),
    LoryConfig("tail_T64", B=3, L=256, T=64, d=128, d_ff=4096, E=17, dtype="bf16", seed=102),
    LoryConfig("tail_T192", B=1, L=2688, T=192, d=320, d_ff=4032, E=3, dtype="bf16", seed=103),
    LoryConfig("tail_wide", B=2, L=1024, T=256, d=2880, d_ff=192, E=3, dtype="bf16", seed=104),
    # one whole round and four tiles
    LoryConfig("tail_whole_T64", B=1, L=4160, T=64, d=1024, d_ff=1536, E=17, dtype="bf16", seed=115),
    LoryConfig("tail_whole_T128", B=5, L=1664, T=128, d=1024, d_ff=384, E=3, dtype="bf16", seed=116),
    LoryConfig("tail_whole_T192", B=5, L=2496, T=192, d=1024, d_ff=384, E=3, dtype="bf16", seed=117),
]


@pytest.mark.parametrize("cfg", TAIL_CASES, ids=lambda c: c.name)
def test_bf16_ring_gemm_cut_last_round(cfg):
    t = make_inputs(cfg, structured=True)
    got = run_layer(cfg, t)
    compare(cfg, got, oracle_layer(cfg, t, got["w_used"]), ALL, TOL["bf16"])
    saved = run_layer(cfg, t, merged_save=True)
    for key in ALL:
        assert np.array_equal(got[key], saved[key]), key


def test_dense_block_cut_last_round():
    cfg = LoryConfig("dense_tail", B=2, L=2048, T=2048, d=768, d_ff=4160, E=2, dtype="bf16", seed=105)
    print(f"[gpu] {cfg}", flush=True)
    t = make_inputs(cfg, with_dy=False)
    Wbar = torch.stack([to_dev(t[k], cfg).reshape(2, -1) for k in ("Wg", "Wu", "Wd")]).contiguous()
    X = to_dev(t["X"], cfg)
    shape = lb.make_shape(2, cfg.L, cfg.L, cfg.d, cfg.d_ff, 1, X.dtype)
    need = lb.lory_workspace_bytes(shape, lb.LORY_PASS_DENSE)
    assert need > cfg.tokens * cfg.d_ff * 2
    ref = orc.ffn_fwd(t["X"], np.eye(2), t["Wg"], t["Wu"], t["Wd"], cfg.L)["Y"]
    # with the reported workspace, and with one that holds the activation alone
    for size in (need, cfg.tokens * cfg.d_ff * 2):
        ws = torch.full((size + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        Y = torch.full_like(X, float("nan"))
        rc = lb.lib().lory_dense_ffn_fwd(ctypes.byref(shape), X.data_ptr(), Wbar.data_ptr(), Y.data_ptr(), ws.data_ptr(),
                                         size, torch.cuda.current_stream().cuda_stream)
        assert rc == lb.LORY_OK, lb.status_string(rc)
        torch.cuda.synchronize()
        assert bool((ws[size:] == 0x5A).all())
        check(f"{size} bytes", host(Y), ref, TOL["bf16"])


# One whole round before four to eight tiles of 128, 192 and 256 rows, with one source and with the two terms of a ragged
# block's activation.  The reference is the product in fp32 on the same operands.
@pytest.mark.parametrize("B,n_tok,d,d_ff", [
    (65, 128, 1024, 1024), (65, 192, 1024, 1024), (65, 256, 1024, 1024), (66, 100, 1024, 1408), (66, 180, 1024, 1024),
])
def test_dense_block_cut_round_after_a_whole_one(B, n_tok, d, d_ff):
    print(f"[gpu] dense_tail {B} {n_tok} {d} {d_ff}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(105)
    X = torch.randn((B, n_tok, d), generator=gen, device="cuda").bfloat16()
    Wbar = torch.stack([torch.randn((B, d * d_ff), generator=gen, device="cuda").mul_(0.02).bfloat16() for _ in range(3)])
    ref = []
    for b in range(B):
        wg, wu, wd = (Wbar[i, b].float().reshape((d, d_ff) if i < 2 else (d_ff, d)) for i in range(3))
        x = X[b].float()
        ref.append((torch.nn.functional.silu(x @ wg) * (x @ wu)) @ wd)
    ref = host(torch.stack(ref))
    shape = lb.make_shape(B, n_tok, n_tok, d, d_ff, 1, X.dtype)
    need, act = lb.lory_workspace_bytes(shape, lb.LORY_PASS_DENSE), B * n_tok * d_ff * (2 if n_tok % 64 == 0 else 4)
    assert need > act
    got = {}
    # with the reported workspace, with more, and (where calls take so little) with one that holds the activation alone
    for size in (need, need + (8 << 20)) + ((act,) if n_tok % 64 == 0 else ()):
        ws = torch.full((size + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        Y = torch.full_like(X, float("nan"))
        rc = lb.lib().lory_dense_ffn_fwd(ctypes.byref(shape), X.data_ptr(), Wbar.data_ptr(), Y.data_ptr(), ws.data_ptr(),
                                         size, torch.cuda.current_stream().cuda_stream)
        assert rc == lb.LORY_OK, lb.status_string(rc)
        torch.cuda.synchronize()
        assert bool((ws[size:] == 0x5A).all())
        got[size] = Y
        check(f"{size} bytes", host(Y), ref, TOL["bf16"])
    assert torch.equal(got[need], got[need + (8 << 20)])


def test_bf16_recompute_bf16_grads_and_accumulate(default_budget):
    cfg = BF16_CASES[0][0]
    lb.lory_set_slab_budget(1 << 20)
    t = make_inputs(cfg, structured=True)
    w1 = make_routing_weights(cfg, "peaked")
    # no saved activations: the backward recomputes G and U; gradients stored as bf16
    got = run_layer(cfg, t, w_override=w1, save=False, grad_dtype=torch.bfloat16)
    ref = oracle_layer(cfg, t, w1)
    compare(cfg, got, ref, ("Y", "dX", "dWg", "dWu", "dWd", "dw"), TOL["bf16"])
    X, Wg, Wu, Wd, dY = (to_dev(t[k], cfg) for k in ("X", "Wg", "Wu", "Wd", "dY"))
    w = torch.from_numpy(w1).cuda()
    for gd in (torch.float32, torch.bfloat16):
        base = [torch.full(Wg.shape, 0.5, dtype=gd, device="cuda"),
                torch.full(Wu.shape, -0.25, dtype=gd, device="cuda"),
                torch.full(Wd.shape, 2.0, dtype=gd, device="cuda")]
        lb.lory_merged_ffn_bwd(X, w, Wg, Wu, Wd, dY, cfg.T, dWg=base[0], dWu=base[1], dWd=base[2],
                               accumulate=True, grad_dtype=gd)
        torch.cuda.synchronize()
        for got_sum, c, key in ((base[0], 0.5, "dWg"), (base[1], -0.25, "dWu"), (base[2], 2.0, "dWd")):
            # the increment itself is held to the bf16 bar; a bf16 sum c + dW is stored with one more
            # rounding, uniform within half a bf16 spacing (<= 2^-7 |c + dW|), i.e. an rms error of at
            # most 2^-7 / sqrt(12) of the stored values, measured here against the increment
            rms = lambda a: float(np.sqrt(np.mean(np.square(a))))
            store = (2.0 ** -7 / np.sqrt(12.0)) * rms(ref[key] + c) / rms(ref[key]) if gd == torch.bfloat16 else 0.0
            err = rel_l2(host(got_sum) - c, ref[key])
            print(f"[parity] accumulate {key} {gd}: {err:.2e} (bar {TOL['bf16'] + store:.2e})", flush=True)
            assert err <= TOL["bf16"] + store, (key, gd, err)


def test_bf16_onehot_and_determinism(default_budget):
    cfg = BF16_CASES[0][0]
    lb.lory_set_slab_budget(1 << 20)
    t = make_inputs(cfg)
    w1 = make_routing_weights(cfg, "onehot")
    a = run_layer(cfg, t, w_override=w1)
    b = run_layer(cfg, t, w_override=w1)
    ref = oracle_layer(cfg, t, w1)
    compare(cfg, a, ref, ALL, TOL["bf16"])
    for key in ALL:
        assert np.array_equal(a[key], b[key]), key


@pytest.mark.parametrize("idx", [0, 6])
def test_bf16_saved_merged_parameters_match_remerge(idx, default_budget):
    """The forward may hand its merged parameters to the backward; results are those of the
    re-merging path (same values, same accumulation order), and within tolerance of the oracle."""
    cfg, budget = BF16_CASES[idx]
    lb.lory_set_slab_budget(budget)
    t = make_inputs(cfg, structured=True)
    a = run_layer(cfg, t, merged_save=True)
    b = run_layer(cfg, t, merged_save=False)
    ref = oracle_layer(cfg, t, a["w_used"])
    compare(cfg, a, ref, ALL, TOL["bf16"])
    for key in ALL:
        assert np.array_equal(a[key], b[key]), key


# ------------------------------------------------------------------ merge inside the GEMM

FUSED_CASES = [
    # T = 256: one segment per wavefront; odd number of 64-column blocks, K not a multiple of 64
    LoryConfig("fused_T256", B=2, L=1024, T=256, d=192, d_ff=320, E=8, dtype="bf16", seed=91),
    # T = 128 with more than 16 experts: the four-wave kernel on the large tile (two segments per wavefront); with at most 16
    # the eight-wave kernel, like the T = 64 cases below
    LoryConfig("fused_T128", B=2, L=512, T=128, d=128, d_ff=192, E=32, dtype="bf16", seed=92),
    LoryConfig("fused_T128_small", B=1, L=512, T=128, d=128, d_ff=128, E=5, dtype="bf16", seed=93),
    # T = 64: three tasks along the rows
    LoryConfig("fused_T64", B=3, L=512, T=64, d=128, d_ff=256, E=16, dtype="bf16", seed=94),
    # T = 64 on the eight-wave kernel with the second group of eight experts partly and wholly absent
    LoryConfig("fused_T64_E11", B=2, L=256, T=64, d=128, d_ff=192, E=11, dtype="bf16", seed=97),
    LoryConfig("fused_T64_E5", B=1, L=512, T=64, d=64, d_ff=128, E=5, dtype="bf16", seed=98),
    # T = 64 with more than 16 experts: the four-wave kernel, two segments per wavefront
    LoryConfig("fused_T64_E32", B=1, L=512, T=64, d=64, d_ff=128, E=32, dtype="bf16", seed=99),
    # the eight-wave kernel with a row chunk that the tokens do not fill: one segment alone, one beyond a whole chunk, and
    # one beyond the eight chunks that share an XCD's L2, with more gate/up tasks than workgroups
    LoryConfig("fused_T64_one_segment", B=1, L=64, T=64, d=64, d_ff=64, E=3, dtype="bf16", seed=120),
    LoryConfig("fused_T64_rows_over", B=3, L=192, T=64, d=192, d_ff=320, E=13, dtype="bf16", seed=121),
    LoryConfig("fused_T128_rows_over", B=5, L=256, T=128, d=192, d_ff=320, E=11, dtype="bf16", seed=126),
    LoryConfig("fused_T64_many", B=5, L=832, T=64, d=256, d_ff=1536, E=9, dtype="bf16", seed=122),
    LoryConfig("fused_one_expert", B=1, L=1024, T=256, d=64, d_ff=64, E=1, dtype="bf16", seed=95),
    # more tasks than one round of workgroups per XCD block, several K steps per source
    LoryConfig("fused_many_tasks", B=4, L=2048, T=128, d=512, d_ff=1024, E=16, dtype="bf16", seed=96),
    # the small tile of the four-wave kernel
    LoryConfig("fused_T128_small_E17", B=1, L=512, T=128, d=128, d_ff=128, E=17, dtype="bf16", seed=133),
    # many tasks on the four-wave kernel, with more than 16 experts and with the forms for at most 16
    LoryConfig("fused_many_tasks_E20", B=4, L=2048, T=128, d=512, d_ff=1024, E=20, dtype="bf16", seed=134),
    LoryConfig("fused_many_tasks_T256", B=4, L=2048, T=256, d=512, d_ff=1024, E=12, dtype="bf16", seed=135),
]


@pytest.fixture
def fused_everywhere():
    lb.lory_set_fused_merge(2)
    yield
    lb.lory_set_fused_merge(1)


@pytest.mark.parametrize("cfg", FUSED_CASES, ids=lambda c: c.name)
@pytest.mark.parametrize("save", [True, False], ids=["saved_GU", "recompute_GU"])
def test_bf16_fused_merge_gemm(cfg, save, fused_everywhere, default_budget):
    """Token contractions with the merge inside the GEMM (no merged parameter in memory), forward
    and backward, against the oracle; and bit-reproducible."""
    t = make_inputs(cfg, structured=True)
    got = run_layer(cfg, t, save=save, grad_dtype=torch.bfloat16)
    ref = oracle_layer(cfg, t, got["w_used"])
    names = ALL if save else ("Y", "dX", "dWg", "dWu", "dWd", "dw")
    compare(cfg, got, ref, names, TOL["bf16"])
    again = run_layer(cfg, t, save=save, grad_dtype=torch.bfloat16)
    for key in names:
        assert np.array_equal(got[key], again[key]), key


# Each contraction is merged inside the GEMM or through the slab on its own: long contractions of few segments go through the
# slab, short ones do not.
@pytest.mark.parametrize("d,d_ff,fused,slab", [(64, 704, ("fused_gate_up", "fused_dA"), ("gemm_down", "gemm_dX")),
                                               (704, 64, ("fused_down", "fused_dX"), ("gemm_gate_up", "gemm_dA"))])
@pytest.mark.parametrize("save", [True, False], ids=["saved_GU", "recompute_GU"])
def test_bf16_contractions_choose_for_themselves(d, d_ff, fused, slab, save, default_budget):
    cfg = LoryConfig(f"mixed_{d}", B=3, L=192, T=64, d=d, d_ff=d_ff, E=6, dtype="bf16", seed=125)
    t = make_inputs(cfg, structured=True)
    print(f"[gpu] {cfg}", flush=True)
    lb.lory_profile_enable(True)
    try:
        lb.lory_profile_read()
        got = run_layer(cfg, t, save=save, grad_dtype=torch.bfloat16)
        classes = {s["name"] for s in lb.lory_profile_read()}
    finally:
        lb.lory_profile_enable(False)
    assert classes.issuperset(fused + slab)
    ref = oracle_layer(cfg, t, got["w_used"])
    compare(cfg, got, ref, ALL if save else ("Y", "dX", "dWg", "dWu", "dWd", "dw"), TOL["bf16"])


# The estimate behind the choice counts the merged values that segments share: the first two of every sequence.  Sixteen
# sequences of two 128-token segments go through the slab, one sequence of as many segments is merged inside the GEMM.  A
# forward pass that does not keep G and U counts their fp32 planes.  Reference: everything through the slab.
@pytest.mark.parametrize("B,N,d,d_ff,fused,not_kept", [
    (16, 2, 1024, 1408, set(), "gemm_gate_up"), (1, 32, 1024, 1408, {"fused_gate_up", "fused_dA"}, "gemm_gate_up"),
    (20, 2, 768, 1408, {"fused_gate_up", "fused_dA"}, "gemm_gate_up"), (1, 40, 768, 1408, {"fused_gate_up", "fused_dA"}, "fused_gate_up"),
])
def test_bf16_choice_counts_shared_segments(B, N, d, d_ff, fused, not_kept, default_budget):
    print(f"[gpu] shared segments {B} {N} {d} {d_ff}", flush=True)
    T, E, gen = 128, 2, torch.Generator(device="cuda").manual_seed(131)
    rand = lambda *s, sigma=1.0: torch.randn(s, generator=gen, device="cuda").mul_(sigma).bfloat16()
    X, dY, W = rand(B, N * T, d), rand(B, N * T, d), [rand(E, d, d_ff, sigma=0.02), rand(E, d, d_ff, sigma=0.02), rand(E, d_ff, d, sigma=0.02)]
    w = lb.lory_route(X, rand(d, E, sigma=d ** -0.5), T, d_ff=d_ff)
    out = {}
    lb.lory_profile_enable(True)
    try:
        for mode in (0, 1):
            lb.lory_set_fused_merge(mode)
            lb.lory_profile_read()
            G, U = (torch.empty((B * N * T, d_ff), dtype=X.dtype, device="cuda") for _ in range(2))
            Y = lb.lory_merged_ffn_fwd(X, w, *W, T, G_save=G, U_save=U)
            grads = lb.lory_merged_ffn_bwd(X, w, *W, dY, T, G_save=G, U_save=U)
            kept = {s["name"] for s in lb.lory_profile_read()}
            Yn = lb.lory_merged_ffn_fwd(X, w, *W, T)
            classes = {s["name"] for s in lb.lory_profile_read()}
            out[mode] = (Y, Yn) + tuple(grads)
            assert {c for c in kept if c.startswith("fused")} == (fused if mode else set()), kept
            assert classes & {"gemm_gate_up", "fused_gate_up"} == {not_kept if mode else "gemm_gate_up"}, classes
    finally:
        lb.lory_profile_enable(False)
        lb.lory_set_fused_merge(1)
    for i, (a, b) in enumerate(zip(*out.values())):
        check(f"output {i}", host(b), host(a), TOL["bf16"])


# A lowered budget holds less than G and U of all tokens: a forward pass that does not keep them takes the slab, block by
# block, whether its tokens fill the row chunks or not.
@pytest.mark.parametrize("save", [True, False], ids=["saved_GU", "recompute_GU"])
@pytest.mark.parametrize("B,L", [(3, 192), (1, 512)])
def test_bf16_contractions_within_a_lowered_budget(B, L, save, default_budget):
    cfg = LoryConfig("mixed_budget", B=B, L=L, T=64, d=64, d_ff=704, E=6, dtype="bf16", seed=125)
    t = make_inputs(cfg, structured=True)
    print(f"[gpu] {cfg}", flush=True)
    lb.lory_set_slab_budget(1 << 20)
    lb.lory_profile_enable(True)
    try:
        lb.lory_profile_read()
        got = run_layer(cfg, t, save=save, grad_dtype=torch.bfloat16)
        classes = {s["name"] for s in lb.lory_profile_read()}
    finally:
        lb.lory_profile_enable(False)
    assert ("gemm_gate_up" in classes) == (not save) and classes.issuperset(("fused_gate_up", "fused_dA"))
    ref = oracle_layer(cfg, t, got["w_used"])
    compare(cfg, got, ref, ALL if save else ("Y", "dX", "dWg", "dWu", "dWd", "dw"), TOL["bf16"])


# Expert stacks of 2 GiB and more: byte offsets beyond 2^31 on the eight-wave kernel, and stacks that it does not take (4 GiB
# and more), which run on the four-wave kernel where a forward pass keeps G and U.  Reference: everything through the slab.
@pytest.mark.parametrize("T,d,d_ff,E,L,mode", [(64, 4096, 16448, 16, 192, 2), (64, 8192, 32832, 8, 4096, 1), (128, 8192, 32832, 8, 1024, 2)])
def test_bf16_merge_inside_the_gemm_of_very_large_stacks(T, d, d_ff, E, L, mode, default_budget):
    print(f"[gpu] very large stacks {T} {d} {d_ff} {L}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(132)

    def rand(*shape, sigma=1.0):
        out = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
        for part in out:   # one matrix in fp32 at a time
            part.copy_(torch.randn(part.shape, generator=gen, device="cuda") * sigma)
        return out

    def rel(a, b):
        err, ref = 0.0, 0.0
        for x, y in zip(a, b):
            err += float((x.float() - y.float()).square().sum(dtype=torch.float64))
            ref += float(y.float().square().sum(dtype=torch.float64))
        return (err / ref) ** 0.5

    X, dY = rand(1, L, d), rand(1, L, d)
    W = [rand(E, d, d_ff, sigma=0.02), rand(E, d, d_ff, sigma=0.02), rand(E, d_ff, d, sigma=0.02)]
    assert 2 * W[0].numel() >= (1 << 31 if E == 16 else 1 << 32)
    w = torch.softmax(torch.randn((L // T, E), generator=gen, device="cuda"), -1)
    out = {}
    lb.lory_profile_enable(True)
    try:
        for m in (0, mode):
            lb.lory_set_fused_merge(m)
            lb.lory_profile_read()
            G, U = (torch.empty((L, d_ff), dtype=X.dtype, device="cuda") for _ in range(2))
            out[m] = [lb.lory_merged_ffn_fwd(X, w, *W, T, G_save=G, U_save=U)]
            out[m] += lb.lory_merged_ffn_bwd(X, w, *W, dY, T, G_save=G, U_save=U, grad_dtype=torch.bfloat16)
            got = {s["name"] for s in lb.lory_profile_read()}
            assert {c for c in got if c.startswith("fused")} == ({"fused_gate_up", "fused_down", "fused_dA", "fused_dX"} if m else set()), got
        if mode == 1:   # without kept G and U the activation is rounded once, through the slab
            out[1] += [lb.lory_merged_ffn_fwd(X, w, *W, T)]
            out[0] += [out[0][0]]
            assert {"gemm_gate_up", "fused_down"} <= {s["name"] for s in lb.lory_profile_read()}
    finally:
        lb.lory_profile_enable(False)
        lb.lory_set_fused_merge(1)
    for i, (a, b) in enumerate(zip(*out.values())):
        err = rel(b, a)
        print(f"[parity] output {i}: {err:.2e}", flush=True)
        assert err <= TOL["bf16"], i


# Without saved G and U the activation is formed from fp32 and rounded once, as through the slab.  Tensor-wide relative
# rounding errors, 1.65e-3 each: weights of gate and up, activation, weights of down, output.  G and U rounded before would
# add two more of that size (SwiGLU's slopes are near 1): 1.2 times the error; 1.03 allows for the scatter of its parts.
@pytest.mark.parametrize("T", [64, 128])
def test_bf16_fused_activation_rounds_once(T, default_budget):
    cfg = LoryConfig(f"once_T{T}", B=3, L=3 * T, T=T, d=320, d_ff=704, E=6, dtype="bf16", seed=126)
    t = make_inputs(cfg, structured=True)
    ref, err = None, {}
    try:
        for mode in (0, 2):
            lb.lory_set_fused_merge(mode)
            got = run_layer(cfg, t, save=False, grad_dtype=torch.bfloat16)
            ref = ref or oracle_layer(cfg, t, got["w_used"])
            err[mode] = rel_l2(got["Y"], ref["Y"])
    finally:
        lb.lory_set_fused_merge(1)
    print(f"slab {err[0]:.4e}, merged inside the GEMM {err[2]:.4e}", flush=True)
    assert err[2] <= 1.03 * err[0]


@pytest.fixture
def fused_with_gradients():
    lb.lory_set_fused_merge(3)
    yield
    lb.lory_set_fused_merge(1)


# shapes the expert-gradient kernel takes (at most 16 experts, T a multiple of 64, B L / T a multiple
# of 8); the last one has three tiles along each matrix dimension and experts beyond E in the operand
FSG_CASES = [c for c in FUSED_CASES if c.name in ("fused_T256", "fused_T64", "fused_T64_E11", "fused_T64_E5",
                                                  "fused_many_tasks")]


@pytest.mark.parametrize("cfg", FSG_CASES, ids=lambda c: c.name)
@pytest.mark.parametrize("save", [True, False], ids=["saved_GU", "recompute_GU"])
def test_bf16_fused_expert_gradients(cfg, save, fused_with_gradients, default_budget):
    """As above, and with the per-segment weight gradients kept on chip: expert gradients and
    routing-weight gradients from the kernel that forms X_s^T dG_s; bit-reproducible (every wave adds
    its inner products to a slot of its own, and the slots are summed in a fixed order)."""
    assert cfg.E <= 16 and cfg.T % 64 == 0 and cfg.S % 8 == 0
    t = make_inputs(cfg, structured=True)
    got = run_layer(cfg, t, save=save, grad_dtype=torch.bfloat16)
    ref = oracle_layer(cfg, t, got["w_used"])
    names = ALL if save else ("Y", "dX", "dWg", "dWu", "dWd", "dw")
    compare(cfg, got, ref, names, TOL["bf16"])
    again = run_layer(cfg, t, save=save, grad_dtype=torch.bfloat16)
    for key in names:
        assert np.array_equal(got[key], again[key]), key


def test_bf16_fused_expert_gradients_differ_from_slab_path_only_by_rounding(fused_with_gradients, default_budget):
    """The same call with the slab pipeline for the weight stage (mode 2): the two agree to bf16
    rounding, which shows that mode 3 ran another kernel and that both compute the same thing."""
    cfg = FUSED_CASES[3]
    t = make_inputs(cfg, structured=True)
    on_chip = run_layer(cfg, t, grad_dtype=torch.bfloat16)
    lb.lory_set_fused_merge(2)
    slab = run_layer(cfg, t, grad_dtype=torch.bfloat16)
    for key in ("dWg", "dWu", "dWd", "dw"):
        check(f"{cfg.name} {key} on chip vs slab", on_chip[key], slab[key], TOL["bf16"])
    assert any(not np.array_equal(on_chip[k], slab[k]) for k in ("dWg", "dWu", "dWd"))


def test_bf16_fused_onehot_routing(fused_everywhere):
    """One-hot routing weights select exactly one expert: the fused kernel's merged tiles are then
    copies of that expert's (bf16 values pass through the hi + lo weight pair unchanged)."""
    cfg = FUSED_CASES[3]
    t = make_inputs(cfg)
    w1 = make_routing_weights(cfg, "onehot")
    got = run_layer(cfg, t, w_override=w1)
    ref = oracle_layer(cfg, t, w1)
    compare(cfg, got, ref, ALL, TOL["bf16"])


def test_merged_save_unsupported_shapes_are_rejected():
    shape = lb.make_shape(5, 3840, 64, 64, 128, 64, torch.bfloat16)   # S = 300 > 128 at E = 64
    assert lb.lory_merged_save_bytes(shape) == 0
    shape32 = lb.make_shape(2, 512, 128, 64, 256, 4, torch.float32)
    assert lb.lory_merged_save_bytes(shape32) == 0


# ------------------------------------------------------------------ router backward

ROUTE_BWD_CASES = [
    CONFIGS["C1"],
    LoryConfig("f32_ragged_dims", B=3, L=60, T=20, d=50, d_ff=70, E=5, dtype="f32", seed=21),
    LoryConfig("f32_single_segment", B=2, L=48, T=48, d=32, d_ff=96, E=3, dtype="f32", seed=22),
    LoryConfig("f32_max_experts", B=1, L=32, T=8, d=16, d_ff=24, E=64, dtype="f32", seed=24),
    LoryConfig("f32_one_token_segments", B=2, L=6, T=1, d=12, d_ff=20, E=4, dtype="f32", seed=25),
    LoryConfig("f32_many_segments", B=2, L=640, T=4, d=40, d_ff=8, E=6, dtype="f32", seed=26),
    LoryConfig("bf16_route_bwd", B=2, L=512, T=64, d=192, d_ff=64, E=8, dtype="bf16", seed=41),
    LoryConfig("bf16_route_bwd_E33", B=3, L=384, T=128, d=320, d_ff=64, E=33, dtype="bf16", seed=42),
    # more rows to a wavefront than it has in flight, with a remainder (41) and without (32), over several chunks of segments;
    # several blocks of columns, the last one partly filled, with and without 16-byte accesses
    LoryConfig("f32_route_bwd_rows", B=100, L=697, T=41, d=40, d_ff=8, E=6, dtype="f32", seed=43),
    LoryConfig("bf16_route_bwd_rows", B=64, L=832, T=64, d=192, d_ff=64, E=5, dtype="bf16", seed=44),
    LoryConfig("bf16_route_bwd_wide", B=1, L=192, T=64, d=2176, d_ff=64, E=9, dtype="bf16", seed=45),
    LoryConfig("f32_route_bwd_wide", B=2, L=36, T=12, d=1100, d_ff=8, E=48, dtype="f32", seed=46),
    LoryConfig("f32_route_bwd_wide_odd", B=2, L=36, T=12, d=1101, d_ff=8, E=5, dtype="f32", seed=47),
]


@pytest.mark.parametrize("cfg", ROUTE_BWD_CASES, ids=lambda c: c.name)
def test_route_bwd_matches_oracle(cfg):
    """lory_route_bwd against the oracle's router backward, fed the same dw.

    The routing here is peaked (structured inputs) so that the softmax Jacobian is far from
    degenerate; dw is a seeded N(0,1) tensor, not the FFN's, so that the router path is not small.
    """
    print(f"[gpu] route_bwd {cfg}", flush=True)
    t = make_inputs(cfg, structured=True)
    rng = np.random.Generator(np.random.Philox(cfg.seed + 900))
    dw = rng.standard_normal((cfg.S, cfg.E)).astype(np.float32)
    X, R = to_dev(t["X"], cfg), to_dev(t["R"], cfg)
    hbar = torch.empty((cfg.S, cfg.d), dtype=torch.float32, device="cuda")
    w = lb.lory_route(X, R, cfg.T, hbar=hbar, d_ff=cfg.d_ff)
    dw_d = torch.from_numpy(dw).cuda()
    # (1) router path alone: added to zeros
    dX0 = torch.zeros_like(X)
    dR = lb.lory_route_bwd(R, w, hbar, dw_d, dX0, cfg.T, d_ff=cfg.d_ff)
    # (2) added in place to an existing gradient, dR accumulated on top of the first result
    base = to_dev(t["dY"], cfg)
    dX1 = base.clone()
    dR2 = dR.clone()
    lb.lory_route_bwd(R, w, hbar, dw_d, dX1, cfg.T, dR=dR2, accumulate_dR=True, d_ff=cfg.d_ff)
    torch.cuda.synchronize()
    ref = orc.route_bwd(t["X"], t["R"], dw.astype(np.float64), cfg.T)
    tol = 1e-4 if cfg.dtype == "f32" else TOL["bf16"]   # fp32: forward softmax and means are fp32
    if cfg.N == 1:
        assert not ref["dX_add"].any() and not ref["dR"].any()
        assert not host(dX0).any() and not host(dR).any()
        assert torch.equal(dX1, base)
        return
    got = {"dX_add": host(dX0), "dR": host(dR)}
    compare(cfg, got, ref, ("dX_add", "dR"), tol)
    total = host(base) + ref["dX_add"].reshape(host(base).shape)
    compare(cfg, {"dX_total": host(dX1)}, {"dX_total": total}, ("dX_total",), tol)
    np.testing.assert_array_equal(host(dR2), 2.0 * host(dR))
    # rows of the last segment of every sequence get nothing from the router path
    last = host(dX0).reshape(cfg.B, cfg.N, cfg.T, cfg.d)[:, -1]
    assert not last.any()


def test_whole_layer_gradient_fp32():
    """route -> fwd -> bwd -> route_bwd on the GPU against the oracle's whole-layer gradient."""
    cfg = CONFIGS["C1"]
    t = make_inputs(cfg, structured=True)
    X, R = to_dev(t["X"], cfg), to_dev(t["R"], cfg)
    Wg, Wu, Wd = (to_dev(t[k], cfg) for k in ("Wg", "Wu", "Wd"))
    dY = to_dev(t["dY"], cfg)
    hbar = torch.empty((cfg.S, cfg.d), dtype=torch.float32, device="cuda")
    w = lb.lory_route(X, R, cfg.T, hbar=hbar, d_ff=cfg.d_ff)
    lb.lory_merged_ffn_fwd(X, w, Wg, Wu, Wd, cfg.T)
    dX, dWg, dWu, dWd, dw = lb.lory_merged_ffn_bwd(X, w, Wg, Wu, Wd, dY, cfg.T)
    dR = lb.lory_route_bwd(R, w, hbar, dw, dX, cfg.T, d_ff=cfg.d_ff)
    torch.cuda.synchronize()
    ref = orc.layer_bwd(t["X"], t["R"], t["Wg"], t["Wu"], t["Wd"], t["dY"], cfg.T)
    got = {"dX": host(dX), "dR": host(dR), "dWg": host(dWg), "dWu": host(dWu), "dWd": host(dWd)}
    compare(cfg, got, ref, ("dX", "dWg", "dWu", "dWd"), 2e-5)
    compare(cfg, got, ref, ("dR",), DR_TOL["f32"])
    assert np.linalg.norm(ref["dR"]) > 0


# ------------------------------------------------------------------ inference: prompt-only routing

INFER_CASES = [
    # (config of the expert stacks, prompt length, token counts of the generation-phase calls)
    (LoryConfig("inf_f32", B=3, L=40, T=40, d=48, d_ff=72, E=5, dtype="f32", seed=51), 40, (1, 3, 8, 13)),
    (LoryConfig("inf_f32_odd", B=2, L=7, T=7, d=50, d_ff=70, E=4, dtype="f32", seed=52), 7, (1, 9)),
    (LoryConfig("inf_bf16", B=4, L=200, T=200, d=256, d_ff=704, E=8, dtype="bf16", seed=53), 200,
     (1, 2, 8, 11, 64, 192)),
    (LoryConfig("inf_bf16_wide", B=2, L=96, T=96, d=1024, d_ff=2816, E=32, dtype="bf16", seed=54), 96,
     (1, 5, 256)),
    # prompts long enough for the two-stage mean (vector and scalar column paths)
    (LoryConfig("inf_bf16_long", B=3, L=1000, T=1000, d=256, d_ff=320, E=16, dtype="bf16", seed=58), 1000, (1, 4)),
    (LoryConfig("inf_f32_long_odd", B=2, L=300, T=300, d=50, d_ff=36, E=3, dtype="f32", seed=59), 300, (2,)),
]


@pytest.mark.parametrize("cfg,Lp,steps", INFER_CASES, ids=lambda v: v.name if isinstance(v, LoryConfig) else None)
def test_prompt_only_routing_inference(cfg, Lp, steps):
    """lory_prompt_merge + lory_dense_ffn_fwd against the oracle: routing on the mean of the whole
    prompt (route with T = L), merged parameters by the definition, then the merged FFN on new tokens
    (the oracle's ffn_fwd with one segment per sequence and the same routing weights)."""
    print(f"[gpu] infer {cfg}", flush=True)
    t = make_inputs(cfg, structured=True, with_dy=False)
    tol = TOL[cfg.dtype]
    X, R = to_dev(t["X"], cfg), to_dev(t["R"], cfg)
    Wg, Wu, Wd = (to_dev(t[k], cfg) for k in ("Wg", "Wu", "Wd"))
    w, Wbar = lb.lory_prompt_merge(X, R, Wg, Wu, Wd)
    torch.cuda.synchronize()
    ref_w = orc.route(t["X"], t["R"], Lp)["w"]
    got_w = host(w)
    assert rel_l2(got_w, ref_w) <= 1e-5
    # merged parameters against the definition, from the GPU's own routing weights
    D = cfg.d * cfg.d_ff
    Wb = host(Wbar).reshape(3, cfg.B, D)
    for i, k in enumerate(("Wg", "Wu", "Wd")):
        ref = np.einsum("be,en->bn", got_w, t[k].astype(np.float64).reshape(cfg.E, D))
        err = rel_l2(Wb[i], ref)
        print(f"[parity] {cfg.name}: {k}_bar={err:.2e}", flush=True)
        assert err <= (1e-5 if cfg.dtype == "f32" else 4e-3)
    # generation phase: new tokens of several counts, the same merged parameters
    for n_tok in steps:
        rng = np.random.Generator(np.random.Philox(cfg.seed * 1000 + n_tok))
        Xn_host = rng.standard_normal((cfg.B, n_tok, cfg.d)).astype(np.float32)
        if cfg.dtype == "bf16":
            Xn_host = round_to_bf16(Xn_host)
        Xn = to_dev(Xn_host, cfg)
        Y = lb.lory_dense_ffn_fwd(Xn, Wbar, cfg.d_ff)
        torch.cuda.synchronize()
        ref = orc.ffn_fwd(Xn_host, got_w, t["Wg"], t["Wu"], t["Wd"], n_tok)["Y"]
        err = rel_l2(host(Y), ref)
        print(f"[parity] {cfg.name}: {n_tok} tokens Y={err:.2e}", flush=True)
        assert np.isfinite(err) and err <= tol, (cfg.name, n_tok, err)


# One row, the edges of the 64- and 128-row tiles, K slices of different lengths (d / 32 and d_ff / 32 not
# multiples of the slice count), and the smallest widths.  How each case runs (tile heights, K slices) is pinned by
# tests/host_sanitize/abi_driver.cpp.
@pytest.mark.parametrize("B,d,d_ff", [(1, 320, 832), (3, 64, 64), (2, 1088, 2880), (40, 192, 1728)])
@pytest.mark.parametrize("n_tok", [1, 63, 65, 128, 200])
def test_dense_block_split_contractions(B, d, d_ff, n_tok):
    cfg = LoryConfig("dense_block", B=B, L=n_tok, T=n_tok, d=d, d_ff=d_ff, E=B, dtype="bf16", seed=61)
    t = make_inputs(cfg, with_dy=False)
    # sequence b uses "expert" b: the oracle's one-hot routing, and the library's parameter set b
    Wbar = torch.stack([to_dev(t[k], cfg).reshape(B, d * d_ff) for k in ("Wg", "Wu", "Wd")]).contiguous()
    Y = lb.lory_dense_ffn_fwd(to_dev(t["X"], cfg), Wbar, d_ff)
    torch.cuda.synchronize()
    ref = orc.ffn_fwd(t["X"], np.eye(B), t["Wg"], t["Wu"], t["Wd"], n_tok)["Y"]
    check(f"dense B={B} d={d} d_ff={d_ff} tokens={n_tok}", host(Y), ref, TOL["bf16"])


# Token counts other than multiples of 64 (decode steps, ragged blocks) keep the activation in fp32 precision into the
# down projection: what separates the output from the exact one is its own rounding to bf16.  The bound is the error of
# the rounded oracle (1.7e-3) with 3 % for rows whose fp32 sums round the other way; an activation rounded to bf16 is
# 1.4 times as far off.  The shapes split both, one or none of the projections, over tiles of every height (pinned by
# tests/host_sanitize/abi_driver.cpp).
@pytest.mark.parametrize("B,n_tok,d,d_ff", [
    (1, 1, 320, 832), (5, 7, 320, 832), (1, 65, 1664, 2816), (2, 100, 512, 1408), (3, 200, 64, 64),
    (130, 100, 64, 64), (150, 129, 64, 128), (130, 250, 64, 64), (40, 63, 192, 1728), (16, 130, 320, 1408),
    # few rows that the ring GEMM takes: gate/up whole, and cut in 64-row tiles
    (4, 14, 1024, 4160), (130, 11, 64, 704), (6, 40, 1024, 1408),
])
def test_dense_block_rounds_only_its_output(B, n_tok, d, d_ff):
    cfg = LoryConfig("dense_exact", B=B, L=n_tok, T=n_tok, d=d, d_ff=d_ff, E=B, dtype="bf16", seed=62)
    print(f"[gpu] {cfg}", flush=True)
    t = make_inputs(cfg, with_dy=False)
    Wbar = torch.stack([to_dev(t[k], cfg).reshape(B, d * d_ff) for k in ("Wg", "Wu", "Wd")]).contiguous()
    Y = host(lb.lory_dense_ffn_fwd(to_dev(t["X"], cfg), Wbar, d_ff))
    ref = orc.ffn_fwd(t["X"], np.eye(B), t["Wg"], t["Wu"], t["Wd"], n_tok)["Y"]
    rounded = np.linalg.norm(round_to_bf16(ref.astype(np.float32)) - ref)
    err = np.linalg.norm(Y - ref)
    assert err <= 1.03 * rounded, (err / rounded, rounded / np.linalg.norm(ref))


# Streamed weights (up to 16 rows): one row and a full block of rows, half a block of columns, fewer K steps than
# wavefronts, an activation slice at the limit of LDS (K slices forced), many and few sequences, and the first row count
# that the ring GEMM takes.  The bound is that of the test above; the least workspace and the library-held scratch give
# the same bits.
@pytest.mark.parametrize("B,n_tok,d,d_ff", [
    (1, 16, 64, 64), (2, 16, 64, 1088), (3, 9, 1088, 192), (1, 2, 2560, 6144), (17, 16, 128, 320), (1, 16, 64, 12352),
    (300, 1, 64, 192), (2, 17, 320, 832),
    # wavefronts of a down projection with two K steps beside wavefronts with one (10 and 14 steps)
    (1, 3, 64, 320), (40, 2, 64, 448),
    # gate/up alone streamed: each number of row blocks, full and with one row; one K step per wavefront and uneven
    # slices, half a block of columns, several sequences
    (1, 17, 1024, 1088), (1, 32, 1024, 1408), (2, 33, 704, 832), (3, 48, 1344, 320), (1, 49, 2048, 128),
    (2, 63, 1024, 832), (1, 24, 2560, 64),
])
def test_dense_block_of_few_rows(B, n_tok, d, d_ff):
    cfg = LoryConfig("dense_stream", B=B, L=n_tok, T=n_tok, d=d, d_ff=d_ff, E=B, dtype="bf16", seed=64)
    print(f"[gpu] {cfg}", flush=True)
    t = make_inputs(cfg, with_dy=False)
    X = to_dev(t["X"], cfg)
    Wbar = torch.stack([to_dev(t[k], cfg).reshape(B, d * d_ff) for k in ("Wg", "Wu", "Wd")]).contiguous()
    Y = lb.lory_dense_ffn_fwd(X, Wbar, d_ff)
    ref = orc.ffn_fwd(t["X"], np.eye(B), t["Wg"], t["Wu"], t["Wd"], n_tok)["Y"]
    rounded = np.linalg.norm(round_to_bf16(ref.astype(np.float32)) - ref)
    assert np.linalg.norm(host(Y) - ref) <= 1.03 * rounded, (np.linalg.norm(host(Y) - ref) / rounded)
    shape = lb.make_shape(B, n_tok, n_tok, d, d_ff, 1, X.dtype)
    assert lb.lory_workspace_bytes(shape, lb.LORY_PASS_DENSE) <= 16 << 20
    Ys = lb.lory_dense_ffn_fwd_static(X, Wbar, d_ff, torch.full_like(X, float("nan")))
    assert torch.equal(Y, Ys)
    if n_tok > 16:
        return
    # the least workspace that is accepted, and the bytes behind it
    lo, hi = 256, lb.lory_workspace_bytes(shape, lb.LORY_PASS_DENSE)
    ws = torch.full((hi + 4096,), 0x5A, dtype=torch.uint8, device="cuda")

    def call(size):
        Yl = torch.full_like(X, float("nan"))
        rc = lb.lib().lory_dense_ffn_fwd(ctypes.byref(shape), X.data_ptr(), Wbar.data_ptr(), Yl.data_ptr(), ws.data_ptr(),
                                         size, torch.cuda.current_stream().cuda_stream)
        return rc, Yl

    while lo < hi:
        mid = (lo + hi) // 512 * 256
        if call(mid)[0] == lb.LORY_OK:
            hi = mid
        else:
            lo = mid + 256
    ws.fill_(0x5A)
    rc, Yl = call(lo)
    assert rc == lb.LORY_OK and torch.equal(Y, Yl) and bool((ws[lo:] == 0x5A).all())


@pytest.mark.parametrize("d,d_ff", [(64, 64), (256, 512)], ids=["two sources", "split"])
def test_dense_block_activation_at_the_end_of_the_range(d, d_ff):
    """An activation above the largest bf16 but finite in fp32 stays finite; an infinite one stays infinite."""
    X = torch.zeros((1, 2, d), device="cuda")
    W = torch.zeros((3, d * d_ff), device="cuda")
    Wg, Wu = W[0].view(d, d_ff), W[1].view(d, d_ff)
    X[0, 0, :2] = 2.0 ** 32
    X[0, 1, 0] = float("inf")
    Wg[0], Wu[0], Wu[1] = 2.0 ** 32, 2.0 ** 31 * 1.9921875, 2.0 ** 31 * 0.005859375
    W[2] = 2.0 ** -100
    a = 2.0 ** 127 * 1.998046875   # silu(2^64) * u; the largest bf16 is 1.9921875 * 2^127
    Y = lb.lory_dense_ffn_fwd(X.bfloat16(), W.bfloat16().reshape(3, 1, d * d_ff).contiguous(), d_ff).double().cpu()
    assert bool(((Y[0, 0] / (d_ff * a * 2.0 ** -100) - 1).abs() < 2.0 ** -8).all()), Y[0, 0, :4]
    assert bool((Y[0, 1] == float("inf")).all()), Y[0, 1, :4]


# Scratch that holds a part of the rows at a time: the library-held array under long ragged blocks, and the least
# workspace that is accepted (several row blocks with a short last one, blocks of fewer than 64 rows, and one block
# without room for partial sums).  The bytes behind the workspace stay as they were.
@pytest.mark.parametrize("B,n_tok,d,d_ff,least", [
    (1, 50000, 64, 192, 73728), (4, 2001, 256, 704, 4325376), (3, 333, 128, 704, 1622016), (600, 100, 64, 64, 7372800),
    (4, 64, 512, 1408, 720896),
])
def test_dense_block_in_little_scratch(B, n_tok, d, d_ff, least):
    cfg = LoryConfig("dense_scratch", B=B, L=n_tok, T=n_tok, d=d, d_ff=d_ff, E=B, dtype="bf16", seed=63)
    print(f"[gpu] {cfg}", flush=True)
    t = make_inputs(cfg, with_dy=False)
    X = to_dev(t["X"], cfg)
    Wbar = torch.stack([to_dev(t[k], cfg).reshape(B, d * d_ff) for k in ("Wg", "Wu", "Wd")]).contiguous()
    ref = orc.ffn_fwd(t["X"], np.eye(B), t["Wg"], t["Wu"], t["Wd"], n_tok)["Y"]
    shape = lb.make_shape(B, n_tok, n_tok, d, d_ff, 1, X.dtype)
    need = lb.lory_workspace_bytes(shape, lb.LORY_PASS_DENSE)
    assert need <= 16 << 20
    outs = []
    for size in (need, least):
        ws = torch.full((size + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        Y = torch.full_like(X, float("nan"))
        rc = lb.lib().lory_dense_ffn_fwd(ctypes.byref(shape), X.data_ptr(), Wbar.data_ptr(), Y.data_ptr(), ws.data_ptr(),
                                         size, torch.cuda.current_stream().cuda_stream)
        assert rc == lb.LORY_OK, (size, lb.status_string(rc))
        torch.cuda.synchronize()
        assert bool((ws[size:] == 0x5A).all())
        check(f"{size} bytes", host(Y), ref, TOL["bf16"])
        outs.append(Y)
    Y = lb.lory_dense_ffn_fwd_static(X, Wbar, d_ff, torch.full_like(X, float("nan")))
    assert torch.equal(Y, outs[0])


def test_prefill_with_saved_merged_parameters_feeds_decode(default_budget):
    """lory_merged_ffn_fwd with T = L and Wbar_save leaves the same buffer lory_prompt_merge writes."""
    cfg = LoryConfig("inf_prefill", B=2, L=128, T=128, d=128, d_ff=256, E=8, dtype="bf16", seed=55)
    t = make_inputs(cfg, structured=True, with_dy=False)
    X, R = to_dev(t["X"], cfg), to_dev(t["R"], cfg)
    Wg, Wu, Wd = (to_dev(t[k], cfg) for k in ("Wg", "Wu", "Wd"))
    w, Wbar = lb.lory_prompt_merge(X, R, Wg, Wu, Wd)
    w2 = lb.lory_route(X, R, cfg.T, d_ff=cfg.d_ff)
    save = lb.alloc_merged_save(lb.make_shape(cfg.B, cfg.L, cfg.T, cfg.d, cfg.d_ff, cfg.E, X.dtype))
    Y = lb.lory_merged_ffn_fwd(X, w2, Wg, Wu, Wd, cfg.T, Wbar_save=save)
    Yd = lb.lory_dense_ffn_fwd(X, Wbar, cfg.d_ff)
    torch.cuda.synchronize()
    assert torch.equal(w, w2)
    assert torch.equal(save.view(torch.bfloat16), Wbar.reshape(-1))
    assert rel_l2(host(Yd), host(Y)) <= 2e-3   # same GEMM kernels; SwiGLU fused against separate pass


def test_prefix_routing_variant():
    """The paper's prefix-routing ablation (Section 5.1): every segment of a sequence uses the merged
    FFN chosen from the first segment.  On the GPU that is lory_prompt_merge on the first T tokens and
    lory_dense_ffn_fwd over the whole sequence; the oracle is its ffn_fwd with the first segment's
    routing weights repeated for every segment."""
    cfg = LoryConfig("prefix", B=2, L=512, T=128, d=128, d_ff=320, E=8, dtype="bf16", seed=56)
    t = make_inputs(cfg, structured=True, with_dy=False)
    X, R = to_dev(t["X"], cfg), to_dev(t["R"], cfg)
    Wg, Wu, Wd = (to_dev(t[k], cfg) for k in ("Wg", "Wu", "Wd"))
    w, Wbar = lb.lory_prompt_merge(X[:, :cfg.T].contiguous(), R, Wg, Wu, Wd)
    Y = lb.lory_dense_ffn_fwd(X, Wbar, cfg.d_ff)
    torch.cuda.synchronize()
    e0 = orc.route(t["X"][:, :cfg.T], t["R"], cfg.T)["w"]            # [B, E]: first segment on itself
    assert rel_l2(host(w), e0) <= 1e-5
    w_rep = np.repeat(host(w), cfg.N, axis=0)                         # the same row for all N segments
    ref = orc.ffn_fwd(t["X"], w_rep, t["Wg"], t["Wu"], t["Wd"], cfg.T)["Y"]
    err = rel_l2(host(Y), ref)
    print(f"[parity] prefix routing Y={err:.2e}", flush=True)
    assert err <= TOL["bf16"]


def test_step_replayed_from_a_hip_graph_matches_eager(default_budget):
    """bench.py times a captured graph of the step; every replay must reproduce the eager results
    bit for bit (the library enqueues kernels only: no allocation, no synchronisation, no memsets)."""
    cfg = LoryConfig("graph", B=2, L=512, T=128, d=256, d_ff=512, E=8, dtype="bf16", seed=61)
    t = make_inputs(cfg, structured=True)
    X, R = to_dev(t["X"], cfg), to_dev(t["R"], cfg)
    Wg, Wu, Wd = (to_dev(t[k], cfg) for k in ("Wg", "Wu", "Wd"))
    dY = to_dev(t["dY"], cfg)
    shape = lb.make_shape(cfg.B, cfg.L, cfg.T, cfg.d, cfg.d_ff, cfg.E, X.dtype)
    ws_f, ws_b = lb.alloc_workspace(shape, lb.LORY_PASS_FWD), lb.alloc_workspace(shape, lb.LORY_PASS_BWD)
    w = torch.empty((cfg.S, cfg.E), dtype=torch.float32, device="cuda")
    hbar = torch.empty((cfg.S, cfg.d), dtype=torch.float32, device="cuda")
    G = torch.empty((cfg.tokens, cfg.d_ff), dtype=X.dtype, device="cuda")
    U = torch.empty_like(G)
    Wbar = lb.alloc_merged_save(shape)
    Y, dX = torch.empty_like(X), torch.empty_like(X)
    dWg, dWu, dWd = torch.empty_like(Wg), torch.empty_like(Wu), torch.empty_like(Wd)
    dw = torch.empty_like(w)
    dR = torch.empty((cfg.d, cfg.E), dtype=torch.float32, device="cuda")
    outs = (w, hbar, Y, dX, dWg, dWu, dWd, dw, dR)

    def step():
        lb.lory_route(X, R, cfg.T, w=w, hbar=hbar, d_ff=cfg.d_ff)
        lb.lory_merged_ffn_fwd(X, w, Wg, Wu, Wd, cfg.T, Y=Y, G_save=G, U_save=U, workspace=ws_f, Wbar_save=Wbar)
        lb.lory_merged_ffn_bwd(X, w, Wg, Wu, Wd, dY, cfg.T, G_save=G, U_save=U, dX=dX, dWg=dWg, dWu=dWu,
                               dWd=dWd, dw=dw, grad_dtype=X.dtype, workspace=ws_b, Wbar_save=Wbar)
        lb.lory_route_bwd(R, w, hbar, dw, dX, cfg.T, dR=dR, d_ff=cfg.d_ff)

    step()
    torch.cuda.synchronize()
    eager = [o.clone() for o in outs]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for rep in range(3):
        for o in outs:
            o.fill_(float("nan")) if o.dtype.is_floating_point else o.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for o, ref in zip(outs, eager):
            assert torch.equal(o, ref), rep
        step()                      # eager work between replays
        torch.cuda.synchronize()


@pytest.mark.parametrize("cfg", [
    CONFIGS["C1"],
    LoryConfig("autograd_bf16", B=2, L=512, T=128, d=256, d_ff=512, E=8, dtype="bf16", seed=71),
], ids=lambda c: c.name)
def test_autograd_wrapper_matches_oracle_layer_gradient(cfg):
    """paper_2405_03133_amd.autograd.lory_layer under torch.autograd against the oracle's whole-layer
    gradient (FFN path + router path with the stop gradient on the first segment)."""
    from paper_2405_03133_amd.autograd import lory_layer
    t = make_inputs(cfg, structured=True)
    leaves = {k: to_dev(t[k], cfg).requires_grad_(True) for k in ("X", "R", "Wg", "Wu", "Wd")}
    dY = to_dev(t["dY"], cfg)
    y = lory_layer(leaves["X"], leaves["R"], leaves["Wg"], leaves["Wu"], leaves["Wd"], cfg.T)
    (y.float() * dY.float()).sum().backward()
    torch.cuda.synchronize()
    ref = orc.layer_bwd(t["X"], t["R"], t["Wg"], t["Wu"], t["Wd"], t["dY"], cfg.T)
    ref_y = orc.layer_fwd(t["X"], t["R"], t["Wg"], t["Wu"], t["Wd"], cfg.T)["Y"]
    tol = 2e-5 if cfg.dtype == "f32" else TOL["bf16"]
    got = {"Y": host(y), "dX": host(leaves["X"].grad), "dWg": host(leaves["Wg"].grad),
           "dWu": host(leaves["Wu"].grad), "dWd": host(leaves["Wd"].grad), "dR": host(leaves["R"].grad)}
    ref = dict(ref, Y=ref_y)
    compare(cfg, got, ref, ("Y", "dX", "dWg", "dWu", "dWd"), tol)
    compare(cfg, got, ref, ("dR",), DR_TOL[cfg.dtype])


@pytest.mark.parametrize("L,lens", [(96, [96, 1, 37, 64]), (512, [512, 1, 300, 257])], ids=["short", "long"])
def test_prompt_merge_with_prompts_of_different_lengths(L, lens):
    """Padded prompts with a length per sequence: routing on the mean of the first len[b] rows only
    (the oracle routes each sequence on its own, with T = L = len[b]); padding rows hold NaN."""
    cfg = LoryConfig("inf_ragged", B=4, L=L, T=L, d=128, d_ff=192, E=8, dtype="bf16", seed=57)
    t = make_inputs(cfg, structured=True, with_dy=False)
    lens = np.array(lens, dtype=np.int32)
    Xp = t["X"].copy()
    for b, n in enumerate(lens):
        Xp[b, n:] = np.nan
    X, R = to_dev(Xp, cfg), to_dev(t["R"], cfg)
    Wg, Wu, Wd = (to_dev(t[k], cfg) for k in ("Wg", "Wu", "Wd"))
    w, Wbar = lb.lory_prompt_merge(X, R, Wg, Wu, Wd, prompt_len=torch.from_numpy(lens).cuda())
    torch.cuda.synchronize()
    got_w = host(w)
    assert np.isfinite(got_w).all() and torch.isfinite(Wbar.float()).all()
    for b, n in enumerate(lens):
        ref = orc.route(t["X"][b:b + 1, :n], t["R"], int(n))["w"][0]
        assert rel_l2(got_w[b], ref) <= 1e-5, (b, n)
    D = cfg.d * cfg.d_ff
    ref_g = np.einsum("be,en->bn", got_w, t["Wg"].astype(np.float64).reshape(cfg.E, D))
    assert rel_l2(host(Wbar).reshape(3, cfg.B, D)[0], ref_g) <= 4e-3


@pytest.mark.parametrize("dtype,classes", [("bf16", "gemm_gate_up + gemm_down"), ("f32", "dense_skinny")])
def test_bench_decode_mode(dtype, classes, capsys, monkeypatch):
    """bench.py --mode infer: one JSON line whose roofline names the kernel classes that a decode step launches."""
    import json
    import types

    import bench

    cfg = LoryConfig("bench_infer", B=2, L=64, T=64, d=128, d_ff=256, E=4, dtype=dtype, seed=71)
    monkeypatch.setitem(CONFIGS, cfg.name, cfg)
    bench.bench_infer(types.SimpleNamespace(config=cfg.name, warmup=1, steps=2))
    out = json.loads(capsys.readouterr().out.strip().splitlines()[-1])
    assert out["roofline"]["kernel"] == classes
    assert out["value"] > 0 and out["roofline"]["achieved"] > 0 and out["roofline"]["avg_launch_us"] > 0
