"""The training step's gradient of the hidden states as partial products over ranges of the vocabulary: every gradient behind it against
the oracle, on both sides of the rule, in both tile classes and in the whole and the masked-edge form."""
import numpy as np
import pytest

import paper_2204_06514_amd as fax
from helpers import to_np, tol, rel_fro
from test_gpu_train import run_train_step, _walk
from workloads import BlockShape, ModelShape, make_model_inputs
from oracle import transformer as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,S,D,V,ranges", [
    (1, 128, 128, 8192, True),      # one whole tile
    (1, 60, 72, 6001, True),        # one cut tile, the last slab of the vocabulary cut
    (1, 130, 136, 4104, True),      # cut tiles in both directions
    (2, 256, 256, 24576, True),
    (2, 300, 520, 9999, True),
    (1, 128, 128, 1024, False)])    # too short: undivided
def test_hidden_gradient_in_ranges(B, S, D, V, ranges):
    ms = ModelShape(BlockShape(B=B, S=S, D=D, H=D // 8, dh=8, F=D, dtype="bf16", sigma_w=0.05, L=1), V=V, S_max=S)
    sh = ms.blk
    p, tok, lab = make_model_inputs(ms, seed=5, generic=True)
    loss_ref, g_ref, _ = orc.model_loss_and_grads(p, tok, lab, sh.H, sh.dh, sh.gelu, sh.ln_eps)
    fax.fax_timing_enable(1)
    try:
        loss, _, _, _, _, grads = run_train_step(ms, p, tok, lab, update=False)
        names = [r["name"] for r in fax.fax_timing_report(64)]
    finally:
        fax.fax_timing_enable(0)
    assert any(n.endswith("_store_ranges") for n in names) == ranges, names
    assert abs(loss - loss_ref) <= 2e-3 * abs(loss_ref)
    bad = {n: rel_fro(to_np(get(grads)), get(g_ref)) for n, get in _walk(grads)}
    assert all(np.isfinite(e) and e <= tol("bf16") for e in bad.values()), bad
    again = run_train_step(ms, p, tok, lab, update=False)[5]
    for n, get in _walk(grads):   # the ranges are folded in a fixed order
        if n != "tok_emb":        # whose scattered rows add up in any order unless asked otherwise
            assert np.array_equal(to_np(get(again)), to_np(get(grads))), n
