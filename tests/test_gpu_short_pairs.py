"""bf16 weight and input gradient of a layer in one launch of 64 x 64 tiles where a product by itself takes larger ones: contractions of one to
three slabs, sizes below, at and beyond a tile, the two sides of the line."""
import numpy as np
import pytest

import paper_2204_06514_amd as fax
from helpers import run_block, dims_of, err, tol
from oracle import transformer as orc
from workloads import BlockShape, make_block_inputs, PARAM_NAMES

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,S,D,H,dh,F,pairs", [(1, 41, 64, 1, 64, 256, 4), (5, 83, 64, 1, 64, 360, 4), (1, 1, 64, 1, 64, 64, 4), (1, 64, 64, 1, 64, 128, 4),
                                                (3, 43, 72, 2, 40, 136, 4), (8, 512, 64, 1, 64, 256, 0)])
def test_block(B, S, D, H, dh, F, pairs):
    sh = BlockShape(B=B, S=S, D=D, H=H, dh=dh, F=F, dtype="bf16", sigma_w=0.05)
    p, x, dy = make_block_inputs(sh, seed=S, generic=True)
    fax.fax_timing_enable(1)
    try:
        out = run_block(sh, p, x, dy)
        rows = {r["name"]: r["launches"] for r in fax.fax_timing_report(64)}
    finally:
        fax.fax_timing_enable(0)
    assert fax.fax_block_bwd_streams(dims_of(sh)) == 1 and rows.get("gemm_mfma_pair", 0) == pairs, rows
    _, c = orc.block_fwd(x, p, sh.H, sh.dh, sh.gelu, sh.ln_eps)
    dx, g, _ = orc.block_bwd(dy, c, p)
    report = {"dx": err(out["dx"], dx, "bf16"), **{k: err(out["grads"][k], g[k], "bf16") for k in PARAM_NAMES}}
    if S == 1:  # one key: nothing depends on queries and keys, whose gradients are zero
        Hd = sh.Hd
        for k in ("wqkv", "bqkv"):
            got, ref = out["grads"][k].reshape(-1, 3 * Hd)[:, 2 * Hd:], g[k].reshape(-1, 3 * Hd)[:, 2 * Hd:]
            report[k] = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    bad = {k: v for k, v in report.items() if not v <= tol("bf16")}
    assert not bad, (bad, report)
