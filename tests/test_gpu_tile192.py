"""256 x 192 tiles, the class for outputs that whole rounds of larger ones leave CUs idle on: every orientation and epilogue against float64
products of the same operands, each size asserted to take the class."""
import numpy as np
import pytest
import torch

import helpers
import paper_2204_06514_amd as fax
from helpers import DEV
from workloads import BlockShape, make_block_inputs

pytestmark = pytest.mark.gpu


def _takes(ta, tb, M, N, K):
    r = fax.fax_gemm_route(fax.FAX_BF16, ta, tb, M, N, K)
    return (r.form, r.tail, r.tile_m, r.tile_n, r.splits) == (fax.FAX_GEMM_MFMA, 0, 256, 192, 1)


def _close(got, ref, err=2.0 ** -8):
    """one rounding to bf16 (2^-9 relative) of an fp32 sum, twice that elementwise beside a floor for what cancels"""
    got, ref = (torch.as_tensor(t, device=DEV).double() for t in (got, ref))
    assert (got - ref).norm() <= 4e-3 * ref.norm()
    assert ((got - ref).abs() <= err * ref.abs() + 1e-4 * ref.abs().max()).all()


# one slab, two, three and more (the pipeline's prologue), tiles that are no multiple of the walk's groups, a second round
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(16384, 768, 64), (16384, 768, 128), (4096, 3072, 192), (8192, 1152, 320), (4096, 5760, 256)])
def test_products(ta, tb, M, N, K):
    assert _takes(ta, tb, M, N, K)
    g = torch.Generator(device=DEV).manual_seed(M + N + K)
    rnd = lambda *s: torch.randn(*s, generator=g, device=DEV).bfloat16()  # noqa: E731
    A, B, R, bias = rnd(*((K, M) if ta else (M, K))), rnd(*((N, K) if tb else (K, N))), rnd(M, N), rnd(N)
    ref = (A.t() if ta else A).double() @ (B.t() if tb else B).double()
    for res, b in ((None, None), (R, bias)):
        C = torch.full((M + 1, N), 7.0, dtype=torch.bfloat16, device=DEV)
        fax.fax_gemm(fax.FAX_BF16, ta, tb, M, N, K, A, A.shape[1], B, B.shape[1], C, N, bias=b, residual=res, ldr=N if res is not None else 0)
        _close(C[:M], ref if res is None else ref + R.double() + bias.double())
        assert (C[M] == 7.0).all()


# every product of the block with a bf16 output but QKV's is T x 768; the partial sums are second outputs beside a residual
@pytest.mark.parametrize("gelu", ["tanh", "erf"])
@pytest.mark.parametrize("partial", [False, True])
def test_block(gelu, partial):
    sh = BlockShape(B=16, S=1024, D=768, H=1, dh=64, F=768, dtype="bf16", sigma_w=0.05, gelu=gelu)
    assert all(_takes(0, tb, sh.T, 768, k) for tb, k in ((0, 64), (0, 768), (1, 768), (1, 192)))
    p, x, dy = make_block_inputs(sh, seed=3, generic=True)
    out = helpers.run_block(sh, p, x, dy, partial=partial)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV).double()  # noqa: E731
    w = {k: t(helpers.to_np(helpers.to_dev(v, "bf16"))) for k, v in p.items()}
    sv, bw = {k: t(v) for k, v in out["saved"].items() if k != "lse"}, {k: t(v) for k, v in out["bwd"].items()}
    X, DY = (t(helpers.to_np(helpers.to_dev(a, "bf16"))).reshape(sh.T, sh.D) for a in (x, dy))
    attn, mlp = sv["ctx"] @ w["wo"], sv["a"] @ w["w2"]
    _close(sv["x1"], X + attn + w["bo"])
    _close(t(out["y"]).reshape(sh.T, sh.D), sv["x1"] + mlp + w["b2"])
    if partial:
        _close(t(out["p_attn"]).reshape(sh.T, sh.D), attn)
        _close(t(out["p_mlp"]).reshape(sh.T, sh.D), mlp)
    u = (sv["h2"] @ w["w1"] + w["b1"]).requires_grad_(True)
    a = torch.nn.functional.gelu(u, approximate="tanh" if gelu == "tanh" else "none")
    d, = torch.autograd.grad(a.sum(), u)
    _close(sv["a"], a.detach())
    _close(sv["dgelu"], d)
    _close(bw["du"], (DY @ w["w2"].t()) * sv["dgelu"])
    _close(bw["dh2"], bw["du"] @ w["w1"].t())
    _close(bw["dh1"], bw["dqkv"] @ w["wqkv"].t())
