"""The fp32 kernels on the matrix cores at the sizes where they can go wrong: around every tile class, single rows, contractions
that end inside a slab, operands that no 16-byte load fits, head widths around 32, 64, 96 and 128; masked rows that are not finite."""
import numpy as np
import pytest
import torch

import paper_2204_06514_amd as fax
import helpers
from helpers import DEV, to_dev, to_np, rel_max
from oracle import transformer as orc
from workloads import BlockShape, make_block_inputs, PARAM_NAMES

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -24  # one fp32 rounding


def _f32(a):
    return a.astype(np.float32).astype(np.float64)


def _padded(a, rows, cols):
    """The matrix in the corner of a larger one filled with NaN: what a kernel fetched there as a factor would show."""
    buf = torch.full((a.shape[0] + rows, a.shape[1] + cols), float("nan"), dtype=torch.float32, device=DEV)
    buf[:a.shape[0], :a.shape[1]] = to_dev(a, "f32")
    return buf


# M, N, K; in this order the 32 x 32 tiles, the 64 x 64, the 128 x 64 and the 128 x 128
GEMM = [(31, 33, 127), (33, 32, 129), (1, 64, 260), (65, 100, 128), (1, 1, 1), (1000, 1000, 72), (960, 1024, 64), (520, 2052, 33),
        (1100, 1003, 33), (2049, 516, 64), (2047, 4100, 32), (1023, 2052, 97), (2048, 4096, 31)]


@pytest.mark.parametrize("M,N,K", GEMM)
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("pad", [0, 3, 4])  # rows of the operands longer than the product: 3 takes the vector loads away
def test_gemm_f32_tiles_and_edges(M, N, K, ta, tb, pad):
    rng = np.random.default_rng(M + N + K)
    A, B = _f32(rng.standard_normal((K, M) if ta else (M, K))), _f32(rng.standard_normal((N, K) if tb else (K, N)))
    bias, R = _f32(rng.standard_normal(N)), _f32(rng.standard_normal((M, N)))
    Ad, Bd = _padded(A, 1, pad), _padded(B, 1, pad)
    C = torch.full((M + 1, N), 7.0, dtype=torch.float32, device=DEV)
    args = (fax.FAX_F32, ta, tb, M, N, K, Ad, Ad.shape[1], Bd, Bd.shape[1], C, N)
    fax.fax_gemm(*args, bias=to_dev(bias, "f32"), residual=to_dev(R, "f32"), ldr=N)
    a, b = A.T if ta else A, B.T if tb else B
    ref = a @ b
    # K products and sums in any order, then two more sums: at most K + 2 roundings of what the magnitudes add up to
    size = np.abs(a) @ np.abs(b)
    assert (np.abs(to_np(C[:M]) - (ref + bias + R)) <= (K + 2) * EPS * (size + np.abs(bias) + np.abs(R))).all()
    fax.fax_gemm(*args, c_f32=1)
    fax.fax_gemm(*args, c_f32=1, accumulate=1)
    assert (np.abs(to_np(C[:M]) - 2 * ref) <= 2 * (K + 1) * EPS * size).all()
    assert (C[M] == 7.0).all()  # nothing beyond the last row


def _f32_product(ta, tb, A, B):
    """A [M, K], B [K, N] on the device -> the kernel's product, operands stored as asked for."""
    M, K, N = A.shape[0], A.shape[1], B.shape[1]
    a, b = (A.T if ta else A).contiguous(), (B.T if tb else B).contiguous()
    C = torch.empty(M, N, dtype=torch.float32, device=DEV)
    fax.fax_gemm(fax.FAX_F32, ta, tb, M, N, K, a, a.shape[1], b, b.shape[1], C, N)
    return C


# M, N and the tile class that the planner gives them; every K ends inside a slab
SPLIT = [(40, 70, 200, (32, 32)), (520, 2052, 72, (64, 64)), (2000, 1000, 1000, (128, 64)), (2047, 4100, 200, (128, 128))]


@pytest.mark.parametrize("M,N,K,tile", SPLIT)
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0)])
def test_gemm_f32_pieces(M, N, K, tile, ta, tb):
    """The three bf16 pieces of a factor: products of single numbers, sums that are not finite, operands below the pieces' range."""
    r = fax.fax_gemm_route(fax.FAX_F32, ta, tb, M, N, K)
    assert (r.tile_m, r.tile_n) == tile
    g = torch.Generator(device=DEV).manual_seed(M + ta + 2 * tb)
    A, B = (torch.randn(s, generator=g, device=DEV) for s in ((M, K), (K, N)))
    # one contraction index: the product of two numbers, of which the pieces leave out less than 2^-24 and two additions round
    one = _f32_product(ta, tb, A[:, :1].contiguous(), B[:1].contiguous()).double()
    ref = A[:, :1].double() @ B[:1].double()
    assert ((one - ref).abs() <= 3 * EPS * ref.abs()).all()
    # tiny factors: the same bound as for any (K sums and products)
    bound = (K + 2) * EPS * (A.abs().double() @ B.abs().double())
    for sa, sb in ((2.0 ** -120, 2.0 ** 100), (2.0 ** 100, 2.0 ** -120)):
        assert ((_f32_product(ta, tb, A * sa, B * sb).double() / (sa * sb) - A.double() @ B.double()).abs() <= bound).all()
    # infinities against ones (whose pieces are zero but for the first) and zeros, NaN, products that overflow, a number that no first piece holds
    A[2] = 0.0
    A[M // 2, 3], A[1, K - 1], A[M - 1, 0], A[2, 0], A[5, 7] = float("inf"), float("nan"), -float("inf"), 3e38, 3.4e38
    B[3, ::3], B[3, 1::3], B[7, 4] = 1.0, 0.0, -1.0
    B[0, N - 1] = 1.0
    got, ref = _f32_product(ta, tb, A, B), A.double() @ B.double()
    for f in (torch.isnan, torch.isposinf, torch.isneginf):
        assert torch.equal(f(got), f(ref.float())), f
    clean = torch.isfinite(ref.float())
    assert ((got.double() - ref).abs() <= (K + 2) * EPS * (A.abs().double().nan_to_num() @ B.abs().double()))[clean].all()


@pytest.mark.parametrize("M,N,K,tile", SPLIT)
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0)])
def test_gemm_f32_small_numbers_beside_ordinary_ones(M, N, K, tile, ta, tb):
    """Rows, columns and single factors down to the smallest fp32 numbers in tiles that hold ordinary ones: every sum within K roundings of
    its own terms.  And what a row that is not finite has computed again leaves the other rows' bits alone."""
    r = fax.fax_gemm_route(fax.FAX_F32, ta, tb, M, N, K)
    assert (r.tile_m, r.tile_n) == tile
    g = torch.Generator(device=DEV).manual_seed(M + ta + 2 * tb)
    A, B = (torch.randn(s, generator=g, device=DEV) for s in ((M, K), (K, N)))
    even = torch.arange(K, device=DEV) % 2 == 0
    A[1] *= torch.where(even, 2.0 ** -120, 1.0)   # one row of both kinds, whose terms are of a size
    B *= torch.where(even, 2.0 ** 60, 2.0 ** -60)[:, None]
    A[3], A[M - 2] = A[3] * 2.0 ** -120, A[M - 2] * 2.0 ** -140
    B[:, 5], B[:, N - 3] = B[:, 5] * 2.0 ** -100, B[:, N - 3] * 2.0 ** -190
    got, ref = _f32_product(ta, tb, A, B), A.double() @ B.double()
    # (2^-150: half of the smallest number there is, for terms and sums that are smaller)
    bound = (K + 2) * (EPS * (A.abs().double() @ B.abs().double()) + 2.0 ** -150)
    assert ((got.double() - ref).abs() <= bound).all()
    A[7, K // 2], A[M - 5, 0] = float("inf"), float("nan")
    again = _f32_product(ta, tb, A, B)
    rest = torch.ones(M, dtype=torch.bool, device=DEV)
    rest[7], rest[M - 5] = False, False
    assert not torch.isfinite(again[~rest]).any()
    assert torch.equal(again[rest], got[rest])


@pytest.mark.parametrize("M,N", [(40, 70), (520, 2052), (2047, 4100)])
@pytest.mark.parametrize("K", [1, 2, 3])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0)])
def test_gemm_f32_short_contractions(M, N, K, ta, tb):
    g = torch.Generator(device=DEV).manual_seed(M + K)
    A, B = (torch.randn(s, generator=g, device=DEV) for s in ((M, K), (K, N)))
    size = A.abs().double() @ B.abs().double()
    # a multiply-add rounds once, by 2^-24 of its result at most
    assert ((_f32_product(ta, tb, A, B).double() - A.double() @ B.double()).abs() <= K * EPS * size).all()


def test_gemm_f32_without_a_contraction():
    bias = torch.arange(40, dtype=torch.float32, device=DEV)
    C = torch.full((3, 40), 7.0, dtype=torch.float32, device=DEV)
    fax.fax_gemm(fax.FAX_F32, 0, 0, 3, 40, 0, None, 0, None, 40, C, 40, bias=bias)
    assert (C == bias).all()


# every epilogue and the column sums, in small and in larger tiles
@pytest.mark.parametrize("shape", [dict(B=1, S=65, D=68, H=1, dh=36, F=132), dict(B=2, S=520, D=260, H=2, dh=64, F=2052),
                                   dict(B=3, S=333, D=257, H=4, dh=33, F=1030)])
@pytest.mark.parametrize("gelu", ["tanh", "erf"])
def test_block_f32(shape, gelu):
    sh = BlockShape(dtype="f32", sigma_w=0.05, gelu=gelu, **shape)
    p, x, dy = make_block_inputs(sh, seed=1, generic=True)
    out = helpers.run_block(sh, p, x, dy)
    y, c = orc.block_fwd(x, p, sh.H, sh.dh, sh.gelu, sh.ln_eps)
    dx, g, _ = orc.block_bwd(dy, c, p)
    worst = {k: rel_max(a, b) for k, a, b in [("y", out["y"], y), ("dx", out["dx"], dx)] + [(k, out["grads"][k], g[k]) for k in PARAM_NAMES]}
    assert max(worst.values()) <= helpers.TOL_F32, worst


# B, S, H, dh: one and several tiles for each of the four waves, the last one full, nearly empty and nearly full
ATTENTION = [(1, 1, 1, 4), (2, 31, 3, 32), (1, 32, 2, 20), (3, 33, 1, 64), (1, 127, 2, 36), (2, 128, 1, 96), (1, 129, 3, 80),
             (1, 161, 2, 128), (2, 200, 2, 100), (1, 515, 2, 64)]


def _attention(B, S, H, dh, qkv, dctx):
    qd, gd = _padded(qkv.reshape(B * S, -1), 40, 0), _padded(dctx.reshape(B * S, -1), 40, 0)
    ctx = torch.full((B * S + 1, H * dh), 7.0, dtype=torch.float32, device=DEV)
    lse = torch.empty((B, H, S), dtype=torch.float32, device=DEV)
    dq = torch.full((B * S + 1, 3 * H * dh), 7.0, dtype=torch.float32, device=DEV)
    fax.fax_attention_fwd(fax.FAX_F32, B, S, H, dh, qd, ctx, lse)
    fax.fax_attention_bwd(fax.FAX_F32, B, S, H, dh, qd, ctx, lse, gd, dq, torch.empty_like(lse))
    assert (ctx[-1] == 7.0).all() and (dq[-1] == 7.0).all()
    return to_np(ctx[:-1]).reshape(B, S, H, dh), to_np(lse), to_np(dq[:-1]).reshape(B, S, 3, H, dh)


def _reference(B, S, H, dh, qkv, dctx):
    t = torch.from_numpy(qkv.reshape(B, S, 3, H, dh)).requires_grad_(True)
    q, k, v = t.permute(2, 0, 3, 1, 4)
    sc = (q @ k.transpose(-1, -2) / dh ** 0.5).masked_fill(torch.ones(S, S, dtype=torch.bool).triu(1), -float("inf"))
    ctx = (torch.softmax(sc, -1) @ v).permute(0, 2, 1, 3)
    ctx.backward(torch.from_numpy(dctx.reshape(B, S, H, dh)))
    return ctx.detach().numpy(), torch.logsumexp(sc, -1).detach().numpy(), t.grad.numpy()


@pytest.mark.parametrize("B,S,H,dh", ATTENTION)
def test_attention_f32_tiles_and_edges(B, S, H, dh):
    rng = np.random.default_rng(S + dh)
    qkv, dctx = _f32(rng.standard_normal((B, S, 3 * H * dh))), _f32(rng.standard_normal((B, S, H * dh)))
    for got, ref in zip(_attention(B, S, H, dh, qkv, dctx), _reference(B, S, H, dh, qkv, dctx)):
        assert rel_max(got, ref) <= helpers.TOL_F32


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("part", [0, 1, 2])
def test_attention_f32_masked_rows_stay_out(part, bad):
    """A query, key or value that is not finite must not reach what the causal mask keeps it from, inside its tile and out."""
    B, S, H, dh, at = 1, 100, 2, 64, 45
    rng = np.random.default_rng(part)
    qkv, dctx = _f32(rng.standard_normal((B, S, 3, H, dh))), _f32(rng.standard_normal((B, S, H * dh)))
    clean = _attention(B, S, H, dh, qkv, dctx)
    qkv[0, at, part, :, 5] = bad
    got = _attention(B, S, H, dh, qkv, dctx)
    assert np.array_equal(got[0][0, :at], clean[0][0, :at])              # earlier outputs
    assert np.array_equal(got[2][0, :at, 0], clean[2][0, :at, 0])        # earlier dQ
    assert not np.isfinite(got[0][0, at]).all()
    if part == 0:                                                        # a query reaches the keys up to its own position only
        assert np.array_equal(got[2][0, at + 1:, 1:], clean[2][0, at + 1:, 1:])
        assert not np.isfinite(got[2][0, at, 1:]).all()


# V: one short of and one more than a vector, rows shorter than a cache line (D = 12: stored at the next vector instead), many vectors
@pytest.mark.parametrize("V,D,S", [(127, 64, 33), (1001, 64, 65), (37, 12, 20), (4099, 68, 40)])
def test_output_projection_f32_over_a_ragged_vocabulary(V, D, S):
    from test_gpu_train import run_train_step, _dev_params, _walk
    from helpers import dims_of
    from workloads import ModelShape, make_model_inputs
    ms = ModelShape(BlockShape(B=1, S=S, D=D, H=1, dh=D, F=128, dtype="f32", sigma_w=0.05, L=1), V=V, S_max=S)
    sh = ms.blk
    p, tok, lab = make_model_inputs(ms, seed=3, generic=True)
    lab[0, 0], lab[0, -1] = V - 1, 0        # the label in the last, partly filled vector
    loss_ref, g_ref, _ = orc.model_loss_and_grads(p, tok, lab, sh.H, sh.dh, sh.gelu, sh.ln_eps)
    loss, params, _, _, _, grads = run_train_step(ms, p, tok, lab, update=False)
    assert abs(loss - loss_ref) <= 1e-5 * abs(loss_ref)
    bad = {name: rel_max(to_np(get(grads)), get(g_ref)) for name, get in _walk(grads)}
    for name in [n for n in bad if n.endswith("bqkv")]:
        del bad[name]                       # its key third is zero but for rounding
    assert max(bad.values()) <= 1e-5, bad
    md = fax.FaxModelDims(dims_of(sh), sh.L, V, S, 0)
    wsb = fax.fax_eval_workspace_bytes(md)
    ws = torch.full((wsb + 4096,), 255, dtype=torch.uint8, device=DEV)   # NaN wherever a kernel reads what none has written
    out = torch.zeros(4, device=DEV)
    fax.fax_eval_step(md, _dev_params(p, "f32"), torch.from_numpy(tok).to(DEV), torch.from_numpy(lab).to(DEV), out, ws, wsb)
    assert abs(out[0].item() - loss) <= 1e-6 * abs(loss)
    assert (ws[wsb:] == 255).all()


# b2's gradient is the sum of dy's rows.  Of N(0, 1) rows: the last rounding (2^-24 / 3^0.5 at most, rms) and those of sixteen terms a slab,
# whose sums are carried exactly, come to 0.7e-7; a plain sum over the slabs gave 1.8e-7 (2048 rows) and 0.9e-7 (128).
@pytest.mark.parametrize("shape,bar", [(dict(B=4, S=512, D=1024, H=16, dh=64, F=4096), 1.0e-7), (dict(B=1, S=1999, D=264, H=4, dh=64, F=500), 1.0e-7),
                                       (dict(B=2, S=64, D=128, H=4, dh=32, F=512), 0.9e-7)])
def test_bias_gradient_is_as_exact_as_a_pass_of_its_own(shape, bar):
    sh = BlockShape(dtype="f32", sigma_w=0.02, **shape)
    p, x, _ = make_block_inputs(sh, seed=0)
    errs = []
    for seed in range(4):
        dy = _f32(np.random.default_rng(seed).standard_normal(x.shape))
        ref = dy.reshape(-1, sh.D).sum(0)
        errs.append(np.linalg.norm(helpers.run_block(sh, p, x, dy)["grads"]["b2"] - ref) / np.linalg.norm(ref))
    assert np.mean(errs) <= bar, errs


def test_bias_gradient_of_infinities():
    sh = BlockShape(dtype="f32", sigma_w=0.02, B=1, S=200, D=64, H=1, dh=64, F=64)
    p, x, dy = make_block_inputs(sh, seed=0)
    dy = np.array(dy)
    dy.reshape(-1, sh.D)[[3, 150], [1, 2]] = np.inf, np.nan
    b2 = helpers.run_block(sh, p, x, dy)["grads"]["b2"]
    assert np.isposinf(b2[1]) and np.isnan(b2[2]) and np.isfinite(np.delete(b2, [1, 2])).all()
