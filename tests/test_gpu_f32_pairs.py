"""fp32 weight and input gradient of a layer in one launch, and both LayerNorms' folds in one: blocks whose products take every
pairing of the small tile classes, sizes at and beside tile edges, gradients added onto given ones.

Bar: that of the fp32 block (max-norm relative 1e-5 per tensor); with gradients added, one fp32 rounding of the sum more.  And the bits of the same
products in launches of their own."""
import numpy as np
import pytest
import torch

import paper_2204_06514_amd as fax
from oracle import transformer as orc
from workloads import BlockShape, make_block_inputs, PARAM_NAMES
from helpers import DEV, run_block, err, dims_of, to_dev, to_np

pytestmark = pytest.mark.gpu

# T = B S; (weight, input) tile edges of the four layers: FFN out, FFN in, attention out, QKV
SHAPES = [
    (BlockShape(B=1, S=1, D=64, H=1, dh=32, F=128, dtype="f32", sigma_w=0.02), None),
    (BlockShape(B=1, S=65, D=128, H=4, dh=32, F=512, dtype="f32", sigma_w=0.02), [(32, 32), (32, 32), (32, 32), (32, 32)]),
    (BlockShape(B=3, S=100, D=256, H=4, dh=64, F=1024, dtype="f32", sigma_w=0.02), [(32, 64), (32, 32), (32, 32), (32, 32)]),
    (BlockShape(B=1, S=33, D=512, H=8, dh=64, F=2048, dtype="f32", sigma_w=0.02), [(64, 32), (64, 32), (32, 32), (64, 32)]),
    (BlockShape(B=2, S=128, D=512, H=8, dh=64, F=2048, dtype="f32", sigma_w=0.02), [(64, 64), (64, 32), (32, 32), (64, 32)]),
    (BlockShape(B=2, S=300, D=260, H=4, dh=96, F=1000, dtype="f32", sigma_w=0.02), None),
    (BlockShape(B=2, S=37, D=130, H=3, dh=36, F=258, dtype="f32", sigma_w=0.02), None),   # operands in no whole vectors
]


def _classes(sh):
    T, D, Hd, F = sh.T, sh.D, sh.Hd, sh.F
    tile = lambda ta, tb, m, n, k: fax.fax_gemm_route(fax.FAX_F32, ta, tb, m, n, k, ta).tile_m  # noqa: E731
    layers = [((F, D), (T, F, D)), ((D, F), (T, D, F)), ((Hd, D), (T, Hd, D)), ((D, 3 * Hd), (T, D, 3 * Hd))]
    return [(tile(1, 0, w[0], w[1], T), tile(0, 1, *g)) for w, g in layers]


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_block_gradients(i, accumulate):
    sh, classes = SHAPES[i]
    assert fax.fax_block_bwd_streams(dims_of(sh)) == 1
    if classes:
        assert _classes(sh) == classes
    p, x, dy = make_block_inputs(sh, seed=i, generic=True)
    rng = np.random.default_rng(i)
    init = {k: rng.standard_normal(p[k].shape).astype(np.float32).astype(np.float64) for k in PARAM_NAMES} if accumulate else None
    out = run_block(sh, p, x, dy, accumulate=accumulate, grads_init=init)
    _, c = orc.block_fwd(x, p, sh.H, sh.dh, sh.gelu, sh.ln_eps)
    dx, g, it = orc.block_bwd(dy, c, p)
    report = {"dx": err(out["dx"], dx, "f32")}
    for k in ("du", "dh2", "dx1", "dctx", "dqkv", "dh1"):
        report[k] = err(out["bwd"][k], it[k].reshape(-1, it[k].shape[-1]), "f32")
    for k in PARAM_NAMES:
        got = out["grads"][k]
        if accumulate:  # the sum's own rounding, 2^-24 of it, is not the gradient's
            off = np.abs(got - (init[k] + g[k])).max()
            report["d" + k] = max(0.0, off - 2.0 ** -23 * np.abs(init[k] + g[k]).max()) / np.abs(g[k]).max()
        elif k == "bqkv":  # the key third is analytically zero
            report["dbqkv"] = np.abs(got - g[k]).max() / np.abs(g[k]).max()
        else:
            report["d" + k] = err(got, g[k], "f32")
    bad = {k: v for k, v in report.items() if not v <= 1e-5}
    assert not bad, (bad, report)


def _product(ta, tb, a, b):
    """float64 arrays of fp32 values -> their product by fax_gemm."""
    (K, M), N = (a.shape, b.shape[1]) if ta else (a.shape[::-1], b.shape[0])
    c = torch.empty((M, N), dtype=torch.float32, device=DEV)
    fax.fax_gemm(fax.FAX_F32, ta, tb, M, N, K, to_dev(a, "f32"), a.shape[1], to_dev(b, "f32"), b.shape[1], c, N, c_f32=ta)
    return to_np(c)


@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_bits_of_the_products_by_themselves(i):
    sh = SHAPES[i][0]
    p, x, dy = make_block_inputs(sh, seed=i, generic=True)
    fax.fax_timing_enable(1)
    try:
        out = run_block(sh, p, x, dy)
        rows = {r["name"]: r["launches"] for r in fax.fax_timing_report(64)}
    finally:
        fax.fax_timing_enable(0)
    assert rows.get("gemm_f32_pair", 0) == (0 if i == len(SHAPES) - 1 else 4), rows
    s, b, g = out["saved"], out["bwd"], out["grads"]
    dy = dy.reshape(sh.T, sh.D)
    for name, act, grad in (("w2", s["a"], dy), ("w1", s["h2"], b["du"]), ("wo", s["ctx"], b["dx1"]), ("wqkv", s["h1"], b["dqkv"])):
        assert np.array_equal(g[name], _product(1, 0, act, grad)), name
    for name, grad, w in (("dh2", b["du"], "w1"), ("dctx", b["dx1"], "wo"), ("dh1", b["dqkv"], "wqkv")):
        assert np.array_equal(b[name], _product(0, 1, grad, p[w])), name
