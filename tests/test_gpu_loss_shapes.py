"""Cross-entropy over rows that end inside a 16-byte vector, at the workgroup shapes they take: one vector, a few, most threads idle, up to and
beyond eight vectors a thread, the most that registers hold."""
import numpy as np
import pytest

from helpers import to_np, rel_fro
from oracle import transformer as orc
from test_gpu_train import run_train_step
from workloads import BlockShape, ModelShape, make_model_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,V", [("bf16", v) for v in (9, 1001, 2051, 16387, 32003, 65529, 65539, 131069)] + [("f32", v) for v in (5, 1001, 32763, 32771, 65533)])
def test_padded_rows(dtype, V):
    ms = ModelShape(BlockShape(B=1, S=24, D=64, H=1, dh=64, F=128, dtype=dtype, sigma_w=0.05, L=1), V=V, S_max=24)
    sh = ms.blk
    p, tok, lab = make_model_inputs(ms, seed=9, generic=True)
    lab[0, 0], lab[0, -1] = V - 1, 0        # the label in the last, partly filled vector
    loss_ref, g_ref, _ = orc.model_loss_and_grads(p, tok, lab, sh.H, sh.dh, sh.gelu, sh.ln_eps)
    loss, _, _, _, _, grads = run_train_step(ms, p, tok, lab, update=False)
    # a loss of bf16 logits: 2^-9 of a logit each, averaged; gradients: the bars of the two types
    assert abs(loss - loss_ref) <= (1e-5 if dtype == "f32" else 1e-3) * abs(loss_ref)
    assert rel_fro(to_np(grads["tok_emb"]), g_ref["tok_emb"]) <= (1e-5 if dtype == "f32" else 2e-2)


@pytest.mark.parametrize("dtype,V", [("bf16", 14890), ("bf16", 20001), ("bf16", 32003), ("f32", 5003)])
def test_padded_rows_on_a_full_chip(dtype, V):
    """Beyond two rows to a CU some lengths take a smaller workgroup: 320 threads instead of 960, 640 as with few rows, 512 instead of 1024, 320 instead of
    640."""
    ms = ModelShape(BlockShape(B=1, S=520, D=64, H=1, dh=64, F=128, dtype=dtype, sigma_w=0.05, L=1), V=V, S_max=520)
    sh = ms.blk
    p, tok, lab = make_model_inputs(ms, seed=9, generic=True)
    lab[0, 0], lab[0, -1] = V - 1, 0
    loss_ref, g_ref, _ = orc.model_loss_and_grads(p, tok, lab, sh.H, sh.dh, sh.gelu, sh.ln_eps)
    loss, _, _, _, _, grads = run_train_step(ms, p, tok, lab, update=False)
    assert abs(loss - loss_ref) <= (1e-5 if dtype == "f32" else 1e-3) * abs(loss_ref)
    assert rel_fro(to_np(grads["tok_emb"]), g_ref["tok_emb"]) <= (1e-5 if dtype == "f32" else 2e-2)


@pytest.mark.parametrize("V", [1001, 32003])
def test_gradients_of_far_off_logits(V):
    """One position, every logit chosen: what an exponential below 2^-126 leaves in the gradient, down to the smallest bf16 number."""
    ms = ModelShape(BlockShape(B=1, S=1, D=64, H=1, dh=64, F=128, dtype="bf16", sigma_w=0.05, L=1), V=V, S_max=1)
    p, tok, lab = make_model_inputs(ms, seed=9, generic=True)
    up = 2.0 ** 20  # the last LayerNorm gives (2^20, 0, ...) whatever comes in
    p["lnf_g"], p["lnf_b"] = np.zeros(64), np.where(np.arange(64) == 0, up, 0.0)
    z = -((np.arange(V) * 7 % 241) / 2.0)   # 0, -0.5, ... -120
    p["tok_emb"] = np.zeros((V, 64))
    p["tok_emb"][:, 0] = z / up
    tok[:], lab[:] = 0, 1
    _, _, _, _, _, grads = run_train_step(ms, p, tok, lab, update=False)
    got = to_np(grads["tok_emb"])[2:, 0] / up
    want = (np.exp(z) / np.exp(z).sum())[2:]
    # one rounding to 8 bits (2^-8 of the power of two below, among subnormals half of 2^-133) of a value that an exponential, a sum and a division have rounded
    assert (np.abs(got - want) <= (2.0 ** -8 + 1e-6) * want + 2.0 ** -134).all()
