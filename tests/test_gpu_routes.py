"""The bf16 product kernels at sizes that the launch planner really gives them, each asserted: contractions cut into ranges and folded (whole,
masked-edge and small tiles), every tile class of the masked-edge form over several slabs, and a layer's two gradients in one launch."""
import numpy as np
import pytest
import torch

import paper_2204_06514_amd as fax
import helpers
from helpers import DEV, to_dev, to_np, rel_max, rel_fro
from oracle import transformer as orc
from workloads import BlockShape, make_block_inputs, round_to_bf16, PARAM_NAMES

pytestmark = pytest.mark.gpu
WHOLE, EDGE, SMALL = fax.FAX_GEMM_MFMA, fax.FAX_GEMM_EDGE, fax.FAX_GEMM_SMALL


def _route(ta, tb, M, N, K, c_f32=0, scratch=0):
    r = fax.fax_gemm_route(fax.FAX_BF16, ta, tb, M, N, K, c_f32, scratch)
    return r.form, r.tile_m, r.tile_n, r.splits


def _weight_grads(sh, out, dy):
    """name -> (activation, gradient) of the block's four weight gradients, as the kernels read them."""
    sv, bw = out["saved"], out["bwd"]
    return {"w2": (sv["a"], dy.reshape(sh.T, sh.D)), "w1": (sv["h2"], bw["du"]), "wo": (sv["ctx"], bw["dx1"]), "wqkv": (sv["h1"], bw["dqkv"])}


BIAS = {"w2": "b2", "w1": "b1", "wo": "bo", "wqkv": "bqkv"}


# Weight gradients in K ranges: (form, tile rows) of the one named, which has to be split.  Whole tiles; the masked-edge form, the last
# range of which ends inside a slab; both small tiles, likewise; outputs whose fold ends inside a vector.
@pytest.mark.parametrize("shape,name,route", [
    (dict(B=8, S=1024, D=1024, H=4, dh=64, F=1024), "w1", (WHOLE, 128)),
    (dict(B=1, S=6001, D=392, H=2, dh=64, F=784), "w1", (EDGE, 128)),
    (dict(B=3, S=1334, D=136, H=2, dh=72, F=136), "w2", (SMALL, 64)),
    (dict(B=3, S=1334, D=360, H=2, dh=64, F=360), "w1", (SMALL, 128)),
    (dict(B=8, S=1024, D=256, H=4, dh=64, F=512), "wo", (SMALL, 64))])
def test_split_contractions(shape, name, route):
    sh = BlockShape(dtype="bf16", sigma_w=0.02, **shape)
    p, x, dy = make_block_inputs(sh, seed=5, generic=True)
    init = {k: np.random.default_rng(1).standard_normal(p[k].shape) * 0.5 for k in PARAM_NAMES}
    out = helpers.run_block(sh, p, x, dy)
    more = helpers.run_block(sh, p, x, dy, accumulate=True, grads_init=init)
    grads = _weight_grads(sh, out, dy)
    form, tile_m, _, splits = _route(1, 0, grads[name][0].shape[1], grads[name][1].shape[1], sh.T, 1, 1)
    assert (form, tile_m) == route and splits > 1
    for k, (act, grad) in grads.items():
        # fp32 sums of exact products: 2^-24 a step, relative to the largest element of a long sum
        assert rel_max(out["grads"][k].reshape(act.shape[1], -1), act.T @ grad) <= 1e-5, k
        assert rel_max(out["grads"][BIAS[k]].reshape(-1), grad.sum(0)) <= 1e-5, k
    for k in PARAM_NAMES:
        ref = init[k].astype(np.float32).astype(np.float64) + out["grads"][k]
        assert rel_max(more["grads"][k], ref) <= 1e-6, k      # the same sums, one more addition


# The masked-edge form, two slabs and more, whole and cut at the end, in each of its tile classes and orientations.
EDGE_PRODUCTS = [(0, 0, 3000, 1200, 1200, 128, 128), (0, 1, 3000, 1200, 4800, 128, 128), (0, 0, 3001, 744, 2984, 128, 128),
                 (0, 0, 3108, 1536, 512, 256, 128), (0, 0, 1200, 4800, 3000, 256, 128), (0, 1, 1999, 4000, 1000, 256, 128),
                 (0, 0, 3000, 4800, 1200, 256, 256), (0, 1, 3001, 2984, 744, 256, 256), (0, 1, 3000, 4800, 128, 256, 256)]


@pytest.mark.parametrize("ta,tb,M,N,K,tile_m,tile_n", EDGE_PRODUCTS)
def test_masked_edge_classes(ta, tb, M, N, K, tile_m, tile_n):
    assert _route(ta, tb, M, N, K) == (EDGE, tile_m, tile_n, 1)
    rng = np.random.default_rng(M + N + K)
    A, B = round_to_bf16(rng.standard_normal((M, K))), round_to_bf16(rng.standard_normal((N, K) if tb else (K, N)))
    R = None if tb else round_to_bf16(rng.standard_normal((M, N)))
    C = torch.full((M + 1, N), 7.0, dtype=torch.bfloat16, device=DEV)
    fax.fax_gemm(fax.FAX_BF16, ta, tb, M, N, K, to_dev(A, "bf16"), K, to_dev(B, "bf16"), B.shape[1], C, N,
                 residual=None if tb else to_dev(R, "bf16"), ldr=0 if tb else N)
    ref = A @ (B.T if tb else B) + (0.0 if tb else R)
    # one rounding to bf16 (2^-9 relative) of an fp32 sum
    assert rel_fro(to_np(C[:M]), ref) <= 4e-3
    assert np.abs(to_np(C[:M]) - ref).max() <= 2 ** -8 * np.abs(ref).max()
    assert (C[M] == 7.0).all()


@pytest.mark.parametrize("M,N,K,tile_m", [(1200, 4800, 3000, 128), (1000, 4000, 1999, 128), (4360, 4104, 200, 256)])
def test_masked_edge_weight_gradients(M, N, K, tile_m):
    assert _route(1, 0, M, N, K, 1) == (EDGE, tile_m, tile_m, 1)
    rng = np.random.default_rng(M + N + K)
    A, B = round_to_bf16(rng.standard_normal((K, M))), round_to_bf16(rng.standard_normal((K, N)))
    C = torch.full((M + 1, N), 7.0, dtype=torch.float32, device=DEV)
    args = (fax.FAX_BF16, 1, 0, M, N, K, to_dev(A, "bf16"), M, to_dev(B, "bf16"), N, C, N)
    ref = A.T @ B
    fax.fax_gemm(*args, c_f32=1)
    assert rel_max(to_np(C[:M]), ref) <= 1e-5
    fax.fax_gemm(*args, c_f32=1, accumulate=1)
    assert rel_max(to_np(C[:M]), 2 * ref) <= 1e-5
    assert (C[M] == 7.0).all()


# Its GELU and GELU' epilogues and fused bias gradients: tile of the feed-forward's forward product (and of the gradient through it)
@pytest.mark.parametrize("shape,tile", [(dict(B=1, S=1999, D=1000, H=15, dh=64, F=4000), (256, 128)),
                                        (dict(B=3, S=1001, D=744, H=12, dh=64, F=2984), (256, 256)),
                                        (dict(B=2, S=1500, D=1200, H=3, dh=80, F=1200), (128, 128))])
@pytest.mark.parametrize("gelu", ["tanh", "erf"])
def test_block_on_masked_edge_classes(shape, tile, gelu):
    sh = BlockShape(dtype="bf16", sigma_w=0.02, gelu=gelu, **shape)
    assert _route(0, 0, sh.T, sh.F, sh.D) == (EDGE, *tile, 1) and _route(0, 1, sh.T, sh.F, sh.D) == (EDGE, *tile, 1)
    assert tile == (128, 128) or _route(1, 0, sh.D, sh.F, sh.T, 1, 1) == (EDGE, 128, 128, 1)
    p, x, dy = make_block_inputs(sh, seed=6, generic=True)
    out = helpers.run_block(sh, p, x, dy)
    y, c = orc.block_fwd(x, p, sh.H, sh.dh, sh.gelu, sh.ln_eps)
    dx, g, _ = orc.block_bwd(dy, c, p)
    worst = {k: rel_fro(a, b) for k, a, b in [("y", out["y"], y), ("dx", out["dx"], dx)] + [(k, out["grads"][k], g[k]) for k in PARAM_NAMES]}
    assert max(worst.values()) <= helpers.TOL_BF16, worst
    for k, (act, grad) in _weight_grads(sh, out, dy).items():
        assert rel_max(out["grads"][k].reshape(act.shape[1], -1), act.T @ grad) <= 1e-5, k
        assert rel_max(out["grads"][BIAS[k]].reshape(-1), grad.sum(0)) <= 1e-5, k
    if gelu == "tanh":
        init = {k: np.full(p[k].shape, 0.5) for k in PARAM_NAMES}
        more = helpers.run_block(sh, p, x, dy, accumulate=True, grads_init=init)
        for k in PARAM_NAMES:
            assert rel_max(more["grads"][k], 0.5 + out["grads"][k]) <= 1e-6, k


# A layer's weight and input gradient in one launch: the rows of either product's tile, for the feed-forward's output and input
# projection, and how many of the four layers take it.  The same bits as from fax_gemm, a launch each.
@pytest.mark.parametrize("shape,w2,w1,pairs", [
    (dict(B=2, S=256, D=256, H=4, dh=64, F=1024), (64, 64), (64, 64), 4),
    (dict(B=2, S=700, D=136, H=2, dh=64, F=544), (64, 128), (64, 64), 4),
    (dict(B=1, S=300, D=712, H=8, dh=88, F=1424), (128, 64), (128, 64), 4),
    (dict(B=1, S=700, D=520, H=4, dh=128, F=2080), (128, 128), (128, 64), 4),
    (dict(B=2, S=700, D=712, H=8, dh=88, F=1424), (128, 128), (128, 128), 4)])
@pytest.mark.parametrize("gelu,accumulate", [("tanh", False), ("erf", True)])
def test_pairs_of_every_tile(shape, w2, w1, pairs, gelu, accumulate):
    sh = BlockShape(dtype="bf16", sigma_w=0.03, gelu=gelu, **shape)
    T = sh.T
    layers = {"w2": (sh.F, sh.D, w2), "w1": (sh.D, sh.F, w1), "wo": (sh.Hd, sh.D, None), "wqkv": (sh.D, 3 * sh.Hd, None)}
    expected = 0
    for k, n, want in layers.values():
        w, d = _route(1, 0, k, n, T, 1, 1), _route(0, 1, T, k, n)
        expected += w[0] == SMALL and w[3] == 1 and d[0] == SMALL
        if want:
            assert (w[0], w[1], d[0], d[1]) == (SMALL, want[0], SMALL, want[1])
    assert pairs == expected
    p, x, dy = make_block_inputs(sh, seed=3, generic=True)
    init = {k: np.full(p[k].shape, 0.5) for k in PARAM_NAMES} if accumulate else None
    fax.fax_timing_enable(1)
    try:
        out = helpers.run_block(sh, p, x, dy, accumulate=accumulate, grads_init=init, flags=fax.FAX_FLAG_SINGLE_STREAM)
        rows = {r["name"]: r["launches"] for r in fax.fax_timing_report(64)}
    finally:
        fax.fax_timing_enable(0)
    assert rows.get("gemm_mfma_pair", 0) == expected, rows

    def gemm(ta, tb, M, N, K, A, B, f32):
        C = torch.full((M, N), 0.5, dtype=torch.float32 if f32 else torch.bfloat16, device=DEV)
        Ad, Bd = to_dev(A, "bf16"), to_dev(B, "bf16")
        fax.fax_gemm(fax.FAX_BF16, ta, tb, M, N, K, Ad, Ad.shape[1], Bd, Bd.shape[1], C, N, c_f32=f32, accumulate=int(accumulate and f32))
        return to_np(C)

    add = 0.5 if accumulate else 0.0
    for k, (act, grad) in _weight_grads(sh, out, dy).items():
        got = out["grads"][k].reshape(act.shape[1], -1)
        assert np.array_equal(got, gemm(1, 0, act.shape[1], grad.shape[1], T, act, grad, 1)), k
        assert rel_max(got - add, act.T @ grad) <= 1e-5, k
        assert rel_max(out["grads"][BIAS[k]].reshape(-1) - add, grad.sum(0)) <= 1e-5, k
    bw = out["bwd"]
    for name, grad, w in [("dh2", bw["du"], p["w1"]), ("dctx", bw["dx1"], p["wo"]), ("dh1", bw["dqkv"], p["wqkv"])]:
        w = np.asarray(w).reshape(-1, grad.shape[1])
        assert np.array_equal(bw[name], gemm(0, 1, T, w.shape[0], grad.shape[1], grad, w, 0)), name
    # through the stored derivative: one rounding to bf16
    du = (dy.reshape(T, sh.D) @ np.asarray(p["w2"]).T) * out["saved"]["dgelu"]
    assert rel_fro(bw["du"], du) <= 4e-3


def test_timing_report_tells_the_kernels_apart():
    def name(ta, tb, M, N, K, c_f32=0, dtype="bf16"):
        A, B = torch.zeros((K, M) if ta else (M, K), dtype=helpers.TDTYPE[dtype], device=DEV), torch.zeros((N, K) if tb else (K, N), dtype=helpers.TDTYPE[dtype], device=DEV)
        C = torch.empty((M, N), dtype=torch.float32 if c_f32 else helpers.TDTYPE[dtype], device=DEV)
        fax.fax_timing_enable(1)
        try:
            fax.fax_gemm(helpers.CODE[dtype], ta, tb, M, N, K, A, A.shape[1], B, B.shape[1], C, N, c_f32=c_f32)
            rows = fax.fax_timing_report(8)
        finally:
            fax.fax_timing_enable(0)
        assert len(rows) == 1
        return rows[0]["name"]

    assert name(0, 0, 4096, 4096, 256) == "gemm_mfma_Ak_Bm_store"
    assert name(0, 0, 3000, 4800, 1200) == "gemm_edge_Ak_Bm_store"
    assert name(0, 1, 512, 256, 1024) == name(0, 1, 500, 264, 1000) == "gemm_mfma_Ak_Bk_store_small"
    assert name(1, 0, 512, 512, 3108, 1) == "gemm_mfma_Am_Bm_f32out_small"
    assert name(0, 0, 500, 500, 500) == "gemm_scalar_Ak_Bm_store"
    assert name(0, 0, 500, 500, 500, dtype="f32") == "gemm_mfma32_Ak_Bm_store"


# Weight gradients of a layer in one launch: how many such launches a backward pass makes.  All four on 256 x 256 tiles; the feed-forward's
# and attention's two, whole tiles; the feed-forward's two on 256 x 256 and attention's on 128 x 128, masked edges; the former alone, 128 x 128; attention's
# two beyond 92 us, apart; the feed-forward's two, each of whole rounds of 256 x 256 tiles, too.
@pytest.mark.parametrize("shape,groups", [
    (dict(B=8, S=1024, D=1024, H=16, dh=64, F=4096), 1),
    (dict(B=8, S=512, D=1024, H=16, dh=64, F=4096), 2),
    (dict(B=3, S=1000, D=1200, H=15, dh=80, F=4800), 2),
    (dict(B=4, S=777, D=512, H=8, dh=64, F=2048), 1),
    (dict(B=11, S=768, D=1024, H=8, dh=128, F=4096), 1),
    (dict(B=14, S=1024, D=1024, H=8, dh=128, F=4096), 0)])
def test_grouped_weight_gradients(shape, groups):
    sh = BlockShape(dtype="bf16", sigma_w=0.03, **shape)
    p, x, dy = make_block_inputs(sh, seed=4, generic=True)

    def run(**kw):
        fax.fax_timing_enable(1)
        try:
            out = helpers.run_block(sh, p, x, dy, **kw)
            rows = {r["name"]: r["launches"] for r in fax.fax_timing_report(64)}
        finally:
            fax.fax_timing_enable(0)
        assert rows.get("gemm_mfma_group", 0) == groups, rows
        return out

    out = run()
    for k, (act, grad) in _weight_grads(sh, out, dy).items():
        # fp32 sums of exact products: 2^-24 a step, relative to the largest element of a long sum
        assert rel_max(out["grads"][k].reshape(act.shape[1], -1), act.T @ grad) <= 1e-5, k
        assert rel_max(out["grads"][BIAS[k]].reshape(-1), grad.sum(0)) <= 1e-5, k
    one = run(flags=fax.FAX_FLAG_SINGLE_STREAM)
    more = run(accumulate=True, grads_init={k: np.full(p[k].shape, 0.5) for k in PARAM_NAMES})
    for k in PARAM_NAMES:
        assert np.array_equal(one["grads"][k], out["grads"][k]), k
        assert rel_max(more["grads"][k], 0.5 + out["grads"][k]) <= 1e-6, k
    assert np.array_equal(one["dx"], out["dx"])
