"""The erf-form GELU of the bf16 product epilogues: the coefficients as they stand in the kernel's source, against math.erfc (CPU only)."""
import math
import os
import re

import numpy as np

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2204_06514_amd", "csrc", "gemm_mfma_kernel.h")
F = np.float32


def _coefficients():
    """-> factor of |u| in 1 / t, factor of u^2 in the exponent, the polynomial's coefficients from the highest, the density's factor."""
    body = open(SRC).read().split("void gelu_erf_both")[1].split("\n}\n")[0]
    num = [float(x) for x in re.findall(r"-?\d+\.\d+(?=f)", body)]
    assert len(num) == 11, num
    return num[0], num[1], num[2:10], num[10]


def _horner(t, poly, mul_add):
    q = np.full_like(t, poly[0])
    for c in poly[1:]:
        q = mul_add(q, t, c)
    return q


def test_polynomial():
    a, b, poly, density = _coefficients()
    x = np.linspace(0.0, 9.5, 20001)
    t = 1.0 / (1.0 + a * math.sqrt(2.0) * x)
    half_erfcx = np.array([math.exp(v * v) * math.erfc(v) / 2 for v in x])
    err = np.abs(_horner(t, poly, lambda q, t, c: q * t + c) * t / half_erfcx - 1.0)
    assert err.max() < 1.07e-7 and err.argmax() == 0, err.max()    # at x = 0 the coefficients add up to 0.499999947
    assert abs(b + 0.5 * math.log2(math.e)) < 1e-8 and abs(density - 1 / math.sqrt(2 * math.pi)) < 1e-8


def test_value_and_derivative_in_fp32():
    a, b, poly, density = _coefficients()
    u = np.linspace(-13.0, 13.0, 40001).astype(F)
    fma = lambda p, q, r: (p.astype(np.float64) * np.asarray(q, np.float64) + np.asarray(r, np.float64)).astype(F)  # noqa: E731
    t = (F(1) / fma(np.abs(u), F(a), F(1))).astype(F)
    e = np.exp2(((u * u).astype(F) * F(b)).astype(np.float64)).astype(F)
    c = ((_horner(t, [F(k) for k in poly], fma) * t).astype(F) * e).astype(F)
    cdf = np.where(u < 0, c, F(1) - c).astype(F)
    g, dg = u * cdf, fma((u * F(density)).astype(F), e, cdf)
    U = u.astype(np.float64)
    phi = np.array([0.5 * math.erfc(-v / math.sqrt(2.0)) for v in U])
    rel = np.abs(g - U * phi) / np.where(U == 0, 1.0, np.abs(U * phi))
    # 2^-24 is 6e-8: eight rounded steps around 1/2, and in the lower tail the rounding of the exponent, u^2 / 2 half units of it
    assert rel[np.abs(u) <= 3].max() < 6e-7 and rel[u >= -9].max() < 4.5e-6, (rel[np.abs(u) <= 3].max(), rel[u >= -9].max())
    assert np.abs(dg - (phi + U * density * np.exp(-U * U / 2))).max() < 3e-7
