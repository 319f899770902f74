"""The small-tile GEMM for products that leave CUs idle, at the sizes where it can go wrong: fewer slabs than its pipeline is deep,
exactly as many and more, contractions that end inside a slab, one short of a tile and one over, both tile shapes."""
import numpy as np
import pytest
import torch

import paper_2204_06514_amd as fax
import helpers
from helpers import DEV, to_dev, to_np, rel_max, rel_fro
from oracle import transformer as orc
from workloads import BlockShape, make_block_inputs, round_to_bf16, PARAM_NAMES

pytestmark = pytest.mark.gpu


def _guarded(a):
    """Rows of NaN behind the matrix: what a kernel fetched there as a factor would show."""
    buf = torch.full((a.shape[0] + 64, a.shape[1]), float("nan"), dtype=torch.bfloat16, device=DEV)
    buf[:a.shape[0]] = to_dev(a, "bf16")
    return buf


# one to eleven slabs of 64, the last one whole or not: 64 x 64 tiles, then 128 x 64
K_SMALL = [8, 64, 72, 128, 136, 192, 256, 264, 320, 384, 448, 704]
SHAPES = [(64, 64, k) for k in K_SMALL] + [(63, 72, 200), (65, 136, 328), (1, 8, 512), (500, 256, 1024)] + \
         [(1537, 512, k) for k in (8, 64, 192, 256, 320, 392, 704)] + [(1920, 640, 1024), (3100, 328, 520)]


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("tb", [0, 1])
def test_deep_gemm_bf16_outputs(M, N, K, tb):
    rng = np.random.default_rng(M + N + K)
    A = round_to_bf16(rng.standard_normal((M, K)))
    B = round_to_bf16(rng.standard_normal((N, K) if tb else (K, N)))
    bias, R = round_to_bf16(rng.standard_normal(N)), round_to_bf16(rng.standard_normal((M, N)))
    C = torch.full((M + 1, N), 7.0, dtype=torch.bfloat16, device=DEV)
    fax.fax_gemm(fax.FAX_BF16, 0, tb, M, N, K, _guarded(A), K, _guarded(B), B.shape[1], C, N, bias=to_dev(bias, "bf16"),
                 residual=None if tb else to_dev(R, "bf16"), ldr=0 if tb else N)
    ref = A @ (B.T if tb else B) + bias + (0.0 if tb else R)
    # one rounding to bf16 (2^-9 relative) of an fp32 sum
    assert rel_fro(to_np(C[:M]), ref) <= 4e-3
    assert np.abs(to_np(C[:M]) - ref).max() <= 2 ** -8 * np.abs(ref).max()
    assert (C[M] == 7.0).all()


@pytest.mark.parametrize("M,N,K", [(64, 64, k) for k in (1, 63, 64, 65, 256, 257, 321)] + [(72, 200, 777), (512, 512, 3108), (1200, 1200, 3000)])
def test_deep_gemm_weight_gradient(M, N, K):
    rng = np.random.default_rng(M + N + K)
    A, B = round_to_bf16(rng.standard_normal((K, M))), round_to_bf16(rng.standard_normal((K, N)))
    C = torch.full((M + 1, N), 7.0, dtype=torch.float32, device=DEV)
    args = (fax.FAX_BF16, 1, 0, M, N, K, _guarded(A), M, _guarded(B), N, C, N)
    fax.fax_gemm(*args, c_f32=1)
    assert rel_max(to_np(C[:M]), A.T @ B) <= 1e-5
    fax.fax_gemm(*args, c_f32=1, accumulate=1)
    assert rel_max(to_np(C[:M]), 2 * (A.T @ B)) <= 1e-5
    assert (C[M] == 7.0).all()


# every epilogue and the bias gradients inside the weight gradients
@pytest.mark.parametrize("shape", [dict(B=2, S=256, D=256, H=4, dh=64, F=1024), dict(B=3, S=100, D=200, H=2, dh=72, F=520),
                                   dict(B=2, S=700, D=328, H=3, dh=64, F=1000)])
@pytest.mark.parametrize("gelu", ["tanh", "erf"])
def test_block_on_deep_tiles(shape, gelu):
    sh = BlockShape(dtype="bf16", sigma_w=0.03, gelu=gelu, **shape)
    p, x, dy = make_block_inputs(sh, seed=2, generic=True)
    out = helpers.run_block(sh, p, x, dy)
    y, c = orc.block_fwd(x, p, sh.H, sh.dh, sh.gelu, sh.ln_eps)
    dx, g, _ = orc.block_bwd(dy, c, p)
    worst = {k: rel_fro(a, b) for k, a, b in [("y", out["y"], y), ("dx", out["dx"], dx)] + [(k, out["grads"][k], g[k]) for k in PARAM_NAMES]}
    assert max(worst.values()) <= helpers.TOL_BF16, worst


# A layer's weight and input gradient in one launch (small products, one stream): the bits that fax_gemm gives from the same tensors in
# launches of their own.  Whole and cut slabs, gradients stored and added to, layers that pair next to layers that do not
# (test_gpu_routes.py: which do, and 128-row tiles).
@pytest.mark.parametrize("shape", [dict(B=2, S=256, D=256, H=4, dh=64, F=1024), dict(B=1, S=100, D=200, H=2, dh=72, F=520),
                                   dict(B=1, S=1, D=64, H=1, dh=64, F=72), dict(B=1, S=65, D=512, H=8, dh=64, F=2048)])
@pytest.mark.parametrize("accumulate", [False, True])
def test_paired_gradients(shape, accumulate):
    sh = BlockShape(dtype="bf16", sigma_w=0.03, gelu="tanh", **shape)
    p, x, dy = make_block_inputs(sh, seed=3, generic=True)
    init = {k: np.full(p[k].shape, 0.5) for k in PARAM_NAMES} if accumulate else None
    out = helpers.run_block(sh, p, x, dy, accumulate=accumulate, grads_init=init)
    T, sv, bw = sh.T, out["saved"], out["bwd"]

    def gemm(ta, tb, M, N, K, A, B, f32):
        C = torch.full((M, N), 0.5, dtype=torch.float32 if f32 else torch.bfloat16, device=DEV)
        Ad, Bd = to_dev(A, "bf16"), to_dev(B, "bf16")
        fax.fax_gemm(fax.FAX_BF16, ta, tb, M, N, K, Ad, Ad.shape[1], Bd, Bd.shape[1], C, N, c_f32=f32,
                     accumulate=int(accumulate and f32))
        return to_np(C)

    dy2 = dy.reshape(T, sh.D)
    for name, act, grad in [("w2", sv["a"], dy2), ("w1", sv["h2"], bw["du"]), ("wo", sv["ctx"], bw["dx1"]),
                            ("wqkv", sv["h1"], bw["dqkv"])]:
        ref = gemm(1, 0, act.shape[1], grad.shape[1], T, act, grad, 1)
        assert np.array_equal(out["grads"][name].reshape(ref.shape), ref), name
    for name, grad, w in [("dh2", bw["du"], p["w1"]), ("dctx", bw["dx1"], p["wo"]), ("dh1", bw["dqkv"], p["wqkv"])]:
        w = np.asarray(w).reshape(-1, grad.shape[1])
        ref = gemm(0, 1, T, w.shape[0], grad.shape[1], grad, w, 0)
        assert np.array_equal(bw[name], ref), name
    y, c = orc.block_fwd(x, p, sh.H, sh.dh, sh.gelu, sh.ln_eps)
    dx, g, _ = orc.block_bwd(dy, c, p)
    add = 0.5 if accumulate else 0.0
    worst = {k: rel_fro(out["grads"][k] - add, g[k]) for k in PARAM_NAMES}
    worst["dx"] = rel_fro(out["dx"], dx)
    assert max(worst.values()) <= helpers.TOL_BF16, worst
