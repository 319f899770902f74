"""Infinities and NaN: what the causal mask keeps from a query or a key must not reach it as 0 * inf, and what is not masked must come
out as the scalar kernels give it (the form a caller can ask for, with no masked pair in its loops)."""
import numpy as np
import pytest
import torch

import paper_2204_06514_amd as fax
from helpers import DEV, TDTYPE, CODE, to_dev, to_np
from workloads import round_to_bf16

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
