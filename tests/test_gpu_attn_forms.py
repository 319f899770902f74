"""bf16 attention in each of its forms (groups x waves of a workgroup: 1x4, 2x2, 2x4, 4x1; dQ and dK/dV apart and in one launch), at
sequence lengths around a workgroup's rows and the groups' tiles.  The form follows from B H, S and the head width alone; test_attn_routes.py asserts which
one each size takes."""
import numpy as np
import pytest
import torch

import paper_2204_06514_amd as fax
from helpers import DEV

pytestmark = pytest.mark.gpu

CASES = [  # B, S, H, dh
    # up to 64 wide, few heads: one tile to three and more than there are groups, whole and ragged
    (1, 1, 1, 64), (2, 31, 3, 32), (1, 33, 2, 64), (1, 65, 3, 40), (1, 128, 2, 64), (1, 193, 2, 64), (1, 256, 4, 64), (1, 321, 3, 56), (1, 2048, 2, 64),
    # more of them: an odd number of tiles and an even one, one launch and two
    (3, 63, 86, 64), (4, 65, 65, 64), (10, 128, 8, 64), (4, 777, 8, 64), (4, 129, 16, 8),
    (4, 512, 16, 64), (5, 517, 15, 64),
    # a full chip
    (33, 128, 16, 64), (15, 523, 8, 64), (35, 100, 30, 24),
    # wider
    (1, 1, 1, 128), (1, 31, 2, 72), (1, 65, 2, 96), (1, 128, 3, 128), (1, 384, 2, 128), (2, 333, 3, 80), (1, 1111, 2, 104), (6, 300, 10, 128), (5, 640, 6, 128),
    (25, 63, 16, 96), (20, 128, 20, 128), (9, 257, 12, 80), (10, 384, 11, 128),
    (41, 128, 10, 128), (45, 70, 10, 88),
    # 4x1 with a group that has no tile; 2x4 whole and ragged, one group alone and an odd number of tiles; 2x2 in two launches and 1x4 at masked widths
    (1, 129, 3, 64), (1, 150, 2, 40), (10, 256, 10, 128), (8, 257, 10, 80), (5, 129, 25, 96), (3, 250, 18, 80), (3, 250, 18, 104), (40, 70, 10, 104)]


def _reference(qkv, dctx):
    B, S, _, H, dh = qkv.shape
    t = qkv.double().requires_grad_(True)
    q, k, v = (t[:, :, i].permute(0, 2, 1, 3) for i in range(3))
    sc = torch.matmul(q, k.transpose(-1, -2)) / dh ** 0.5
    sc = sc.masked_fill(torch.ones(S, S, dtype=torch.bool, device=qkv.device).triu(1), -float("inf"))
    ctx = torch.matmul(torch.softmax(sc, -1), v).permute(0, 2, 1, 3)
    ctx.backward(dctx.double())
    return ctx.detach(), torch.logsumexp(sc, -1).detach(), t.grad


@pytest.mark.parametrize("B,S,H,dh", CASES)
@pytest.mark.parametrize("spread", [1.0, 6.0])  # 6: peaked rows, whose maximum may come late, in any group
def test_attention_forms(B, S, H, dh, spread):
    g = torch.Generator(device=DEV).manual_seed(S + H)
    rows = B * S
    qkv = torch.full((rows + 40, 3 * H * dh), float("nan"), dtype=torch.bfloat16, device=DEV)  # NaN behind the last row
    qkv[:rows] = (torch.randn((rows, 3 * H * dh), generator=g, device=DEV) * torch.tensor([spread, 1.0, 1.0], device=DEV).repeat_interleave(H * dh)).bfloat16()
    dctx = torch.full((rows + 40, H * dh), float("nan"), dtype=torch.bfloat16, device=DEV)
    dctx[:rows] = torch.randn((rows, H * dh), generator=g, device=DEV).bfloat16()
    ctx = torch.full((rows + 1, H * dh), 7.0, dtype=torch.bfloat16, device=DEV)
    lse = torch.full((B * H * S + 1,), 7.0, dtype=torch.float32, device=DEV)
    delta = torch.full((B * H * S + 1,), 7.0, dtype=torch.float32, device=DEV)
    dqkv = torch.full((rows + 1, 3 * H * dh), 7.0, dtype=torch.bfloat16, device=DEV)
    fax.fax_attention_fwd(fax.FAX_BF16, B, S, H, dh, qkv, ctx, lse)
    fax.fax_attention_bwd(fax.FAX_BF16, B, S, H, dh, qkv, ctx, lse, dctx, dqkv, delta)
    for t in (ctx[-1], lse[-1], delta[-1], dqkv[-1]):
        assert (t == 7.0).all()  # nothing beyond the last row
    rc, rl, rg = _reference(qkv[:rows].view(B, S, 3, H, dh), dctx[:rows].view(B, S, H, dh))
    rel = lambda a, b: ((a.double() - b).norm() / b.norm().clamp_min(1e-30)).item()  # noqa: E731
    # ctx: one rounding to bf16 (2^-9) and, in the whole-tile form, one of the probabilities; the gradients two more (dctx and ctx given)
    assert rel(ctx[:-1].view(B, S, H, dh), rc) <= 4e-3
    assert (lse[:-1].view(B, H, S).double() - rl).abs().max().item() <= 2e-5 * max(1.0, rl.abs().max().item())
    got = dqkv[:-1].view(B, S, 3, H, dh)
    for i in range(3):
        if S > 1 or i == 2:  # (of one key alone, dQ and dK are zero but for rounding)
            assert rel(got[:, :, i], rg[:, :, i]) <= 1e-2, i
    again = torch.empty_like(dqkv)
    fax.fax_attention_bwd(fax.FAX_BF16, B, S, H, dh, qkv, ctx, lse, dctx, again, delta)
    assert torch.equal(again[:-1], dqkv[:-1])  # one writer per row, sums in a fixed order
