"""LayerNorm at the edges of its row lengths per thread count: forward, and backward with and without a residual gradient, against float64."""
import pytest
import torch

import paper_2204_06514_amd as fax

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BF16 = [8, 504, 512, 1024, 1032, 2048, 2056, 4096, 4104, 6144, 6152, 8192, 8200, 12288, 12296, 16384]  # 8 elements a vector
F32 = [4, 252, 256, 512, 516, 1024, 1028, 2048, 2052, 3072, 3076, 4096, 4100, 6144, 6148, 8192]


@pytest.mark.parametrize("rows", [1, 37, 3001])
@pytest.mark.parametrize("dtype,D", [("bf16", d) for d in BF16] + [("f32", d) for d in F32])
def test_layernorm_rows(dtype, D, rows):
    rows = rows if D <= 4104 else min(rows, 1200)
    code, t, es = (fax.FAX_BF16, torch.bfloat16, 2.0 ** -8) if dtype == "bf16" else (fax.FAX_F32, torch.float32, 2.0 ** -24)
    g = torch.Generator(device=DEV).manual_seed(D + rows)
    rnd = lambda *s: torch.randn(*s, generator=g, device=DEV)  # noqa: E731
    x, dh, dres = (rnd(rows, D).to(t) for _ in range(3))
    gamma, beta = (1 + 0.1 * rnd(D)).to(t), (0.1 * rnd(D)).to(t)
    X, DH, G = x.double(), dh.double(), gamma.double()
    mean, var = X.mean(1, keepdim=True), X.var(1, unbiased=False, keepdim=True)
    r = (var + 1e-5).rsqrt()
    xh = (X - mean) * r
    h, mu, rstd = torch.empty_like(x), torch.empty(rows, device=DEV), torch.empty(rows, device=DEV)
    fax.fax_layernorm_fwd(code, rows, D, x, gamma, beta, 1e-5, h, mu, rstd)
    # elementwise: one rounding of the result (bf16: half of the last of 8 bits, 2^-8 of the power of two below) and a few of fp32 sums of up to 16384 terms
    close = lambda a, b, e: ((a.double() - b).abs() <= e * (1 + b.abs())).all()  # noqa: E731
    assert close(mu, mean[:, 0], 1e-6) and close(rstd / r[:, 0].float(), torch.ones(rows, device=DEV, dtype=torch.float64), 1e-6)
    assert close(h, xh * G + beta.double(), es + 4e-6)
    n = fax.fax_layernorm_bwd_workspace_bytes(D)
    ws = torch.full((n,), 255, dtype=torch.uint8, device=DEV)
    g1 = DH * G
    dx_ref = r * (g1 - g1.mean(1, keepdim=True) - xh * (g1 * xh).mean(1, keepdim=True))
    for res, acc in ((dres, 0), (None, 1)):
        dx, dg, db = torch.empty_like(x), torch.full((D,), 0.5, device=DEV), torch.full((D,), 0.5, device=DEV)
        fax.fax_layernorm_bwd(code, rows, D, dh, x, mu, rstd, gamma, res, dx, dg, db, acc, ws, n)
        want = dx_ref + (res.double() if res is not None else 0)
        big = 1 + r.max().item() * (D == 4)  # rows of four have standard deviations far below 1
        assert close(dx, want, (es + 4e-6) * big)
        for got, ref in ((dg, (DH * xh).sum(0)), (db, DH.sum(0))):
            assert close(got - 0.5 * acc, ref, 2.0 ** -24 * 8 * rows ** 0.5 * big + 1e-6)
