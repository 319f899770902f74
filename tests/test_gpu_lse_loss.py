"""The validation loss from the output projection's own tiles, without stored logits: whole tiles, a strip of 128 columns, masked rows,
columns and contractions, parts of 128 columns with nothing in them that counts, infinities and NaN.

Every row of the embedding has one element, a power of two: the logits are exact in bf16, and the training step, which stores them so, has the
same loss but for fp32 rounding in another order (the sum of V exponentials, 2^-22 of it in 64 + 4 + 16 steps, and the logarithm's)."""
import numpy as np
import pytest
import torch

import paper_2204_06514_amd as fax
from helpers import DEV, dims_of
from test_gpu_train import run_train_step, _dev_params
from workloads import BlockShape, ModelShape, make_model_inputs, round_to_bf16

pytestmark = pytest.mark.gpu


def _model(T, D, V, seed, B=1):
    ms = ModelShape(BlockShape(B=B, S=T // B, D=D, H=1, dh=64, F=128, dtype="bf16", sigma_w=0.05, L=1), V=V, S_max=(T // B + 7) // 8 * 8)
    p, tok, lab = make_model_inputs(ms, seed=seed, generic=True)
    n = np.arange(V)
    p["tok_emb"][:] = 0
    p["tok_emb"][n, n % D] = np.where(n // D % 2, -1.0, 1.0) * 2.0 ** (n // D % 5 - 3)
    return ms, p, tok, lab


def _eval(ms, p, tok, lab):
    md = fax.FaxModelDims(dims_of(ms.blk), 1, ms.V, ms.S_max, 0)
    wsb = fax.fax_eval_workspace_bytes(md)
    ws = torch.full((wsb,), 255, dtype=torch.uint8, device=DEV)   # NaN wherever a kernel reads what none has written
    out = torch.zeros(4, device=DEV)
    fax.fax_timing_enable(1)
    try:
        fax.fax_eval_step(md, _dev_params(p, "bf16"), torch.from_numpy(tok).to(DEV), torch.from_numpy(lab).to(DEV), out, ws, wsb)
        names = [r["name"] for r in fax.fax_timing_report(64)]
    finally:
        fax.fax_timing_enable(0)
    fused = "gemm_mfma_Ak_Bk_lse" in names
    assert ("lse_row_loss" in names) == fused and ("cross_entropy" in names) == (not fused)   # every kernel of the loss is in the report
    return out[0].item(), fused


SIZES = [(4096, 64, 4096, 4),      # whole tiles, one slab
         (4096, 128, 4224, 4),     # and a strip
         (4096, 64, 3200, 4),      # 128 columns beyond whole tiles whose tiles fit into the round
         (3000, 200, 8003, 3),     # nothing whole: rows, columns, contraction
         (4001, 72, 3329, 1),      # one column beyond a tile
         (3841, 520, 3200, 1)]     # one row beyond, a part of 128 columns masked out


@pytest.mark.parametrize("T,D,V,B", SIZES)
def test_loss_is_that_of_stored_logits(T, D, V, B):
    ms, p, tok, lab = _model(T, D, V, 3, B)
    lab[0, :4] = [0, V - 1, V - 2, V // 2]
    got, fused = _eval(ms, p, tok, lab)
    assert fused
    ref = run_train_step(ms, p, tok, lab, update=False)[0]
    assert abs(got - ref) <= 2e-6 * abs(ref)


def test_few_tiles_keep_the_stored_logits():
    ms, p, tok, lab = _model(2048, 64, 2048, 5)
    got, fused = _eval(ms, p, tok, lab)
    assert not fused and got == run_train_step(ms, p, tok, lab, update=False)[0]


def test_long_tiles_in_badly_filled_rounds_keep_the_stored_logits():
    ms, p, tok, lab = _model(4096, 2048, 8448, 5)   # 528 tiles of 32 slabs, two rounds and 16
    got, fused = _eval(ms, p, tok, lab)
    assert not fused and got == run_train_step(ms, p, tok, lab, update=False)[0]


# Few columns, whole tiles of them (a strip of 128 alone, one tile) and a part of one, at the fewest row tiles the line asks for and one less; eight
# and seven, whose parts take the logits' place and more.
@pytest.mark.parametrize("T,V,B,fused", [(49152, 128, 24, True), (48896, 128, 191, False), (49152, 256, 24, True), (49152, 72, 24, True), (49151, 101, 23, True),
                                         (48896, 72, 191, False), (49152, 8, 24, True), (49152, 7, 24, False)])
def test_few_columns(T, V, B, fused):
    ms, p, tok, lab = _model(T, 64, V, 6, B)
    lab[0, :2] = [0, V - 1]
    got, was_fused = _eval(ms, p, tok, lab)
    assert was_fused == fused
    ref = run_train_step(ms, p, tok, lab, update=False)[0]
    assert abs(got - ref) <= 2e-6 * abs(ref)


@pytest.mark.parametrize("V", [4096, 4203])
@pytest.mark.parametrize("what", ["dominant", "empty part", "minus inf everywhere else", "far below", "nan", "inf"])
def test_extremes(what, V):
    T, D = 4096, 64
    ms, p, tok, lab = _model(T, D, V, 4, 4)
    p["lnf_g"][:] = 0
    p["lnf_b"][:] = 1   # every hidden state is one: the logits are the embedding's elements
    tok = np.full_like(tok, 300)
    lab = np.full_like(lab, 300)
    z = p["tok_emb"].sum(1)
    inf = float("inf")
    at = {"dominant": {777: 300.0}, "empty part": {n: -inf for n in range(128, 256)}, "minus inf everywhere else": {n: -inf for n in range(V) if n != 300},
          "far below": {n: -2.0 ** 17 for n in range(V)}, "nan": {V - 1: float("nan")}, "inf": {5: inf}}[what]
    for n, v in at.items():
        p["tok_emb"][n, n % D] = z[n] = v
    got, fused = _eval(ms, p, tok, lab)
    assert fused
    if what in ("nan", "inf"):
        assert np.isnan(got)
        return
    top = z.max()
    ref = top + np.log(np.exp(z - top).sum()) - z[300]
    assert abs(got - ref) <= 2e-6 * max(abs(ref), abs(top))   # of the logits' size: what cancels in the difference


@pytest.mark.parametrize("V", [4096, 4203])
@pytest.mark.parametrize("what", ["largest", "least of all", "least but for one", "a part of the least", "2^29", "2^31", "1e12", "-1e12"])
def test_ends_of_the_range(what, V):
    """Logits of 2.5e38 and 3e38 either way, which log2(e) takes beyond fp32's range, and of sizes whose product with it is rounded by 64 and
    more."""
    T, D, big = 4096, 64, 3.0e38
    ms, p, tok, lab = _model(T, D, V, 4, 4)
    p["lnf_g"][:] = 0
    p["lnf_b"][:] = 1   # every hidden state is one: the logits are the embedding's elements
    tok, lab = np.full_like(tok, 300), np.full_like(lab, 300)
    at = {"largest": {300: 2.5e38, 777: 2.5e38}, "least of all": {n: -big for n in range(V)},
          "least but for one": {n: -big if n != 300 else -2.5e38 for n in range(V)}, "a part of the least": {n: -big for n in range(128, 256)},
          "2^29": {n: 1.5 * 2.0 ** 29 for n in (300, 301, 777)}, "2^31": {n: 1.5 * 2.0 ** 31 for n in (300, 301, 777)},
          "1e12": {n: 1.25e12 for n in (300, 301, 777)}, "-1e12": {n: -1.25e12 for n in range(V)}}[what]
    at = {n: round_to_bf16(np.array([v]))[0] for n, v in at.items()}
    z = p["tok_emb"].sum(1)
    for n, v in at.items():
        p["tok_emb"][n, n % D] = z[n] = v
    got, fused = _eval(ms, p, tok, lab)
    assert fused
    ref = np.log(np.exp(z - z.max()).sum()) + (z.max() - z[300])
    assert abs(got - ref) <= 2e-6 * max(1.0, abs(ref))


@pytest.mark.parametrize("V", [4096, 4203])
def test_dominant_labels_cost_nothing_below_zero(V):
    """The label's logit some 300 above the others: its loss is zero whatever order the logits are summed in."""
    T, D = 4096, 520
    rng = np.random.default_rng(7)
    for _ in range(6):
        ms, p, tok, lab = _model(T, D, V, 4, 4)
        p["lnf_g"][:] = 0
        p["lnf_b"][:] = p["tok_emb"][300] = round_to_bf16(rng.standard_normal(D) * 0.8)
        got, fused = _eval(ms, p, tok, np.full_like(lab, 300))
        assert fused and 0.0 <= got <= 1e-4   # 300 in fp32, 2^-15, twice
