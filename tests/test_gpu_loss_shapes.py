"""Cross-entropy over rows that end inside a 16-byte vector, at the workgroup shapes they take: one vector, a few, most threads idle, up to and
beyond eight vectors a thread, the most that registers hold."""
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
