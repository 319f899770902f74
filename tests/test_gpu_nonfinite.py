"""Infinities and NaN: what the causal mask keeps from a query or a key must not reach it as 0 * inf, and what is not masked must come
out as the scalar kernels give it (the form a caller can ask for, with no masked pair in its loops)."""
import numpy as np
import pytest
import torch

import paper_2204_06514_amd as fax
from helpers import DEV, TDTYPE, CODE, dims_of, to_dev, to_np
from test_gpu_train import run_train_step, _dev_params
from workloads import BlockShape, ModelShape, make_model_inputs, round_to_bf16

pytestmark = pytest.mark.gpu
NAN, INF = float("nan"), float("inf")


def _attention(dtype, path, B, S, H, dh, qkv, dctx):
    td = TDTYPE[dtype]
    ctx = torch.full((B, S, H * dh), 7.0, dtype=td, device=DEV)
    lse = torch.full((B, H, S), 7.0, device=DEV)
    dq = torch.full((B, S, 3 * H * dh), 7.0, dtype=td, device=DEV)
    delta = torch.empty_like(lse)
    fax.fax_attention_fwd(CODE[dtype], B, S, H, dh, qkv, ctx, lse, path)
    fax.fax_attention_bwd(CODE[dtype], B, S, H, dh, qkv, ctx, lse, dctx, dq, delta, path)
    return {"ctx": to_np(ctx).reshape(B, S, H, dh), "lse": to_np(lse), "dqkv": to_np(dq).reshape(B, S, 3, H, dh)}


def _same_kind(a, b):
    """NaN where NaN, the same infinity where infinite."""
    return np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(np.where(np.isinf(a), a, 0.0), np.where(np.isinf(b), b, 0.0))


def _agree(got, ref, tol):
    for k in ref:
        assert _same_kind(got[k], ref[k]), (k, np.argwhere(np.isfinite(got[k]) != np.isfinite(ref[k]))[:4])
        ok = np.isfinite(ref[k])
        assert np.linalg.norm(got[k][ok] - ref[k][ok]) <= tol * np.linalg.norm(ref[k][ok]), k


# B, S, H, dh and the position that is not finite: in the last, partly filled tile; in a whole tile; where the last tile's missing rows
# would hold that of an earlier tile; in the first tile of a workgroup's second pass; all three row widths
@pytest.mark.parametrize("B,S,H,dh,at", [(1, 1000, 2, 64, 999), (1, 1000, 2, 80, 600), (2, 200, 1, 128, 130), (1, 330, 8, 64, 200),
                                         (1, 330, 1, 96, 70), (1, 17, 2, 64, 9)])
@pytest.mark.parametrize("part", ["q", "k", "v", "dctx"])
@pytest.mark.parametrize("bad", [NAN, INF, -INF])
def test_bf16_attention_of_any_length(B, S, H, dh, at, part, bad):
    rng = np.random.default_rng(S + dh)
    qkv, dctx = round_to_bf16(rng.standard_normal((B, S, 3, H, dh))), round_to_bf16(rng.standard_normal((B, S, H, dh)))
    if part == "dctx":
        dctx[0, at, :, 5] = bad
    else:
        qkv[0, at, "qkv".index(part), :, 5] = bad
    q, d = to_dev(qkv.reshape(B, S, -1), "bf16"), to_dev(dctx.reshape(B, S, -1), "bf16")
    got = _attention("bf16", fax.PATH_AUTO, B, S, H, dh, q, d)
    ref = _attention("bf16", fax.PATH_SCALAR, B, S, H, dh, q, d)
    assert np.isfinite(ref["ctx"][0, :at]).all() and np.isfinite(ref["dqkv"][0, :at, 0]).all()
    # two roundings to bf16 (2^-9) of the same sums; the gradients also carry those of two ctx, which delta is formed from
    _agree(got, ref, 1e-2)


# The loss over a vocabulary that ends inside a 16-byte vector (first two: with one element, the only one of its thread), and over a
# whole one: a logit that is NaN makes its row's loss and gradient NaN wherever it stands.
@pytest.mark.parametrize("V,col", [(121, 120), (1001, 1000), (1001, 3), (1024, 1019)])
def test_a_nan_logit_reaches_the_loss(V, col):
    ms = ModelShape(BlockShape(B=1, S=64, D=64, H=1, dh=64, F=128, dtype="bf16", sigma_w=0.05, L=1), V=V, S_max=64)
    p, tok, lab = make_model_inputs(ms, seed=1, generic=True)
    last = np.arange(8) + col // 8 * 8
    nan = last[last < V] if V % 8 == 0 else [col]     # all that the thread has
    p["tok_emb"][nan] = NAN
    tok, lab = np.full_like(tok, 1), np.full_like(lab, 2)
    loss, _, _, _, _, grads = run_train_step(ms, p, tok, lab, update=False)
    assert np.isnan(loss)
    # every row's gradient is NaN, the hidden states' with it, and every row of the embedding's
    assert np.isnan(to_np(grads["lnf_g"])).all() and np.isnan(to_np(grads["tok_emb"])[:V]).all()
    md = fax.FaxModelDims(dims_of(ms.blk), 1, V, 64, 0)
    ws = torch.empty(fax.fax_eval_workspace_bytes(md), dtype=torch.uint8, device=DEV)
    out = torch.zeros(4, device=DEV)
    fax.fax_eval_step(md, _dev_params(p, "bf16"), torch.from_numpy(tok).to(DEV), torch.from_numpy(lab).to(DEV), out, ws, ws.numel())
    assert np.isnan(out[0].item())
