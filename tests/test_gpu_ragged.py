"""Kernels for sizes that no tile divides, at the sizes where they can go wrong: one less, exactly and one more than a
tile, single rows, contractions that end inside a slab.  Against float64 products of the same rounded operands."""
import numpy as np
import pytest
import torch

import paper_2204_06514_amd as fax
from helpers import DEV, TDTYPE, CODE, to_dev, to_np, rel_max, rel_fro
from oracle import transformer as orc
from workloads import round_to_bf16

pytestmark = pytest.mark.gpu

# M, N, K.  The masked-edge GEMM and the small-tile one that takes most of these keep what is contiguous in memory a multiple of 8 elements;
# the rest is free.  (test_gpu_routes.py: every tile class of the masked-edge form.)
FORWARD = [(1, 8, 8), (127, 136, 64), (129, 120, 72), (300, 264, 200), (1000, 1160, 136), (20003, 1160, 72)]
WEIGHT_GRAD = [(8, 8, 1), (136, 120, 63), (128, 256, 65), (264, 200, 3001), (4360, 4104, 200)]


@pytest.mark.parametrize("M,N,K", FORWARD)
@pytest.mark.parametrize("tb,res", [(0, False), (0, True), (1, False)])
def test_edge_gemm_bf16_outputs(M, N, K, tb, res):
    rng = np.random.default_rng(M + N + K)
    A = round_to_bf16(rng.standard_normal((M, K)))
    B = round_to_bf16(rng.standard_normal((N, K) if tb else (K, N)))
    bias = round_to_bf16(rng.standard_normal(N))
    R = round_to_bf16(rng.standard_normal((M, N)))
    C = torch.full((M + 1, N), 7.0, dtype=torch.bfloat16, device=DEV)
    fax.fax_gemm(fax.FAX_BF16, 0, tb, M, N, K, to_dev(A, "bf16"), K, to_dev(B, "bf16"), B.shape[1], C, N, bias=to_dev(bias, "bf16"),
                 residual=to_dev(R, "bf16") if res else None, ldr=N if res else 0)
    ref = A @ (B.T if tb else B) + bias + (R if res else 0.0)
    # one rounding to bf16 (2^-9 relative) of an fp32 sum
    assert rel_fro(to_np(C[:M]), ref) <= 4e-3
    assert np.abs(to_np(C[:M]) - ref).max() <= 2 ** -8 * np.abs(ref).max()
    assert (C[M] == 7.0).all()   # nothing beyond the last row


@pytest.mark.parametrize("M,N,K", WEIGHT_GRAD)
def test_edge_gemm_weight_gradient(M, N, K):
    rng = np.random.default_rng(M + N + K)
    A, B = round_to_bf16(rng.standard_normal((K, M))), round_to_bf16(rng.standard_normal((K, N)))
    C = torch.full((M + 1, N), 7.0, dtype=torch.float32, device=DEV)
    args = (fax.FAX_BF16, 1, 0, M, N, K, to_dev(A, "bf16"), M, to_dev(B, "bf16"), N, C, N)
    fax.fax_gemm(*args, c_f32=1)
    assert rel_max(to_np(C[:M]), A.T @ B) <= 1e-5
    fax.fax_gemm(*args, c_f32=1, accumulate=1)
    assert rel_max(to_np(C[:M]), 2 * (A.T @ B)) <= 1e-5
    assert (C[M] == 7.0).all()


def test_edge_gemm_reads_nothing_beyond_the_contraction():
    """Rows of the operands past K hold NaN: a product that fetched one of them as a factor would show it."""
    rng = np.random.default_rng(5)
    M, N, K = 136, 264, 70
    A, B = round_to_bf16(rng.standard_normal((K, M))), round_to_bf16(rng.standard_normal((K, N)))
    Ad = torch.full((K + 64, M), float("nan"), dtype=torch.bfloat16, device=DEV)
    Bd = torch.full((K + 64, N), float("nan"), dtype=torch.bfloat16, device=DEV)
    Ad[:K], Bd[:K] = to_dev(A, "bf16"), to_dev(B, "bf16")
    C = torch.empty((M, N), dtype=torch.float32, device=DEV)
    fax.fax_gemm(fax.FAX_BF16, 1, 0, M, N, K, Ad, M, Bd, N, C, N, c_f32=1)
    assert rel_max(to_np(C), A.T @ B) <= 1e-5


# B, S, H, dh: around the 64-row tiles and 128-row workgroups, head widths around 64, 96 and 128 (and one chunk), one to many heads
ATTENTION = [(1, 1, 1, 8), (2, 17, 3, 64), (1, 63, 8, 80), (3, 64, 1, 128), (1, 65, 2, 96), (2, 127, 2, 72), (1, 128, 2, 32),
             (1, 129, 3, 128), (1, 192, 2, 64), (2, 200, 4, 104), (1, 333, 16, 48), (1, 1000, 2, 80), (1, 777, 2, 64)]


def _guarded(a):
    """The tensor with rows of NaN behind it: what a kernel fetched there as a factor would show."""
    buf = torch.full((a.size + 4096,), float("nan"), dtype=torch.bfloat16, device=DEV)
    buf[:a.size] = to_dev(a, "bf16").reshape(-1)
    return buf[:a.size].view(a.shape)


@pytest.mark.parametrize("B,S,H,dh", ATTENTION)
def test_edge_attention(B, S, H, dh):
    rng = np.random.default_rng(S * 3 + dh)
    Hd = H * dh
    qkv, dctx = round_to_bf16(rng.standard_normal((B, S, 3 * Hd))), round_to_bf16(rng.standard_normal((B, S, Hd)))
    ctx_ref, lse_ref = orc.attention_fwd(qkv, H, dh)
    qd, dd = _guarded(qkv), _guarded(dctx)
    full = lambda n, t: torch.full((n + 1024,), 7.0, dtype=t, device=DEV)  # noqa: E731
    ctx, lse = full(ctx_ref.size, torch.bfloat16), full(lse_ref.size, torch.float32)
    dq, delta = full(qkv.size, torch.bfloat16), full(lse_ref.size, torch.float32)
    fax.fax_attention_fwd(fax.FAX_BF16, B, S, H, dh, qd, ctx, lse, fax.PATH_AUTO)
    fax.fax_attention_bwd(fax.FAX_BF16, B, S, H, dh, qd, ctx, lse, dd, dq, delta, fax.PATH_AUTO)
    for t, n in ((ctx, ctx_ref.size), (lse, lse_ref.size), (dq, qkv.size), (delta, lse_ref.size)):
        assert (t[n:] == 7.0).all()   # nothing written behind the outputs
    # ctx: one rounding to bf16 (2^-9) of an fp32 sum; lse: fp32
    assert rel_fro(to_np(ctx[:ctx_ref.size]).reshape(ctx_ref.shape), ctx_ref) <= 4e-3
    assert np.abs(to_np(lse[:lse_ref.size]).reshape(lse_ref.shape) - lse_ref).max() <= 2e-5
    # the gradients: one rounding each, plus that of ctx, which delta is formed from (the bar of the scalar kernels)
    got, ref = to_np(dq[:qkv.size]).reshape(qkv.shape), orc.attention_bwd(dctx, qkv, H, dh)
    for i in range(3):
        g, r = got[..., i * Hd:(i + 1) * Hd], ref[..., i * Hd:(i + 1) * Hd]
        if S > 1 or i == 2:
            assert rel_fro(g, r) <= 6e-3, i
        else:   # one query, one key: the gradients of Q and K cancel to nothing but the rounding of ctx
            assert np.abs(g - r).max() <= 4e-2


def test_edge_attention_agrees_with_the_plain_form():
    """The same heads with eight more positions, which no earlier query sees: the first 256 rows have to agree."""
    rng = np.random.default_rng(11)
    S, H, dh = 256, 2, 128
    qkv = to_dev(round_to_bf16(rng.standard_normal((1, S + 8, 3 * H * dh))), "bf16")
    ctx = torch.empty((1, S, H * dh), dtype=torch.bfloat16, device=DEV); lse = torch.empty((1, H, S), device=DEV)
    ctx2 = torch.empty((1, S + 8, H * dh), dtype=torch.bfloat16, device=DEV); lse2 = torch.empty((1, H, S + 8), device=DEV)
    fax.fax_attention_fwd(fax.FAX_BF16, 1, S, H, dh, qkv[:, :S].contiguous(), ctx, lse, fax.PATH_MFMA)
    fax.fax_attention_fwd(fax.FAX_BF16, 1, S + 8, H, dh, qkv, ctx2, lse2, fax.PATH_AUTO)
    assert rel_fro(to_np(ctx2[:, :S]), to_np(ctx)) <= 8e-3
    assert np.abs(to_np(lse2[..., :S]) - to_np(lse)).max() <= 2e-5


# V: one short of a tile (127: the padded rows are whole tiles, the embedding is not), one more than a vector, many vectors and a rest
@pytest.mark.parametrize("V,D,S", [(127, 64, 128), (1001, 128, 65), (4099, 64, 128)])
def test_output_projection_over_a_ragged_vocabulary(V, D, S):
    from test_gpu_train import run_train_step, _dev_params, _walk
    from helpers import dims_of
    from workloads import BlockShape, ModelShape, make_model_inputs
    ms = ModelShape(BlockShape(B=1, S=S, D=D, H=1, dh=D, F=128, dtype="bf16", sigma_w=0.05, L=1), V=V, S_max=S)
    sh = ms.blk
    p, tok, lab = make_model_inputs(ms, seed=3, generic=True)
    lab[0, 0], lab[0, -1] = V - 1, 0        # the label in the last, partly filled vector
    loss_ref, g_ref, _ = orc.model_loss_and_grads(p, tok, lab, sh.H, sh.dh, sh.gelu, sh.ln_eps)
    loss, params, _, _, _, grads = run_train_step(ms, p, tok, lab, update=False)
    assert abs(loss - loss_ref) <= 2e-3 * abs(loss_ref)
    bad = {name: rel_fro(to_np(get(grads)), get(g_ref)) for name, get in _walk(grads)}
    # one block of bf16 activations (2^-9 each rounding): the bar of the block and training tests
    assert max(bad.values()) <= 2e-2, bad
    md = fax.FaxModelDims(dims_of(sh), sh.L, V, S, 0)
    wsb = fax.fax_eval_workspace_bytes(md)
    ws = torch.full((wsb + 4096,), 255, dtype=torch.uint8, device=DEV)   # NaN wherever a kernel reads what none has written
    out = torch.zeros(4, device=DEV)
    fax.fax_eval_step(md, _dev_params(p, "bf16"), torch.from_numpy(tok).to(DEV), torch.from_numpy(lab).to(DEV), out, ws, wsb)
    assert abs(out[0].item() - loss) <= 1e-6 * abs(loss)
    assert (ws[wsb:] == 255).all()


# Sums that cancel to about 1e-4 of their terms show the probabilities' own error, which the rounding of the outputs otherwise hides:
# keys in pairs of nearly the same score with opposite V (ctx), queries likewise with opposite dO (dV).  Keys from 64 on
# have no weight, so that the two queries of a pair see the same ones.
@pytest.mark.parametrize("dh", [64, 80, 128])
def test_edge_attention_probabilities_are_fp32(dh):
    rng = np.random.default_rng(dh)
    B, S, H, n = 2, 333, 2, 64
    qkv = rng.standard_normal((B, S, 3, H, dh))
    dctx = np.zeros((B, S, H, dh))
    q, k, v = (qkv[:, :, i] for i in range(3))
    q[:, n + 1::2], k[:, 1::2], v[:, 1::2] = q[:, n:-1:2], k[:, 0:-1:2], -v[:, 0:-1:2]
    q[..., 0], k[..., 0] = 0.0, rng.choice([-1.0, 1.0], (B, S, H))
    q[:, n + 1::2, :, 0] = 2.0 ** -10
    k[..., 1], q[..., 1] = 0.0, 1.0
    k[:, 1::2, :, 1] = 2.0 ** -10
    k[..., 2], q[..., 2] = 0.0, 8.0
    k[:, n:, :, 2] = -128.0
    k[:, 1:n:2, :, 0] = k[:, 0:n:2, :, 0]
    g = rng.standard_normal((B, (S - n) // 2, H, dh))
    dctx[:, n:-1:2], dctx[:, n + 1::2] = g, -g
    qkv, dctx = round_to_bf16(qkv).reshape(B, S, -1), round_to_bf16(dctx).reshape(B, S, -1)
    ctx_ref, lse_ref = orc.attention_fwd(qkv, H, dh)
    dv_ref = orc.attention_bwd(dctx, qkv, H, dh)[..., 2 * H * dh:]
    qd, dd = to_dev(qkv, "bf16"), to_dev(dctx, "bf16")
    ctx, lse = torch.empty((B, S, H * dh), dtype=torch.bfloat16, device=DEV), torch.empty((B, H, S), device=DEV)
    dq, delta = torch.empty_like(qd), torch.empty_like(lse)
    err = {}
    for path in (fax.PATH_SCALAR, fax.PATH_AUTO):
        fax.fax_attention_fwd(fax.FAX_BF16, B, S, H, dh, qd, ctx, lse, path)
        fax.fax_attention_bwd(fax.FAX_BF16, B, S, H, dh, qd, ctx, lse, dd, dq, delta, path)
        err[path] = (rel_fro(to_np(ctx[:, n:]), ctx_ref[:, n:]), rel_fro(to_np(dq[:, :n, 2 * H * dh:]), dv_ref[:, :n]))
    # as close as the scalar kernels' fp32 probabilities, whose last bits (2^-24 of the terms, 1e-3 of the sums) differ from these
    for a, s in zip(err[fax.PATH_AUTO], err[fax.PATH_SCALAR]):
        assert a <= 1.25 * s, err
