"""The GELU forms of the bf16 product epilogues: their constants as they stand in the kernel's source, against float64 (CPU only)."""
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


def _fma(p, q, r):
    return (p.astype(np.float64) * np.asarray(q, np.float64) + np.asarray(r, np.float64)).astype(F)


def _tanh_form(u):
    """The kernel's steps, with the constants as they stand in its source, each rounded to fp32."""
    body = open(SRC).read().split("void gelu_tanh_both")[1].split("\n}\n")[0]
    b, a, d, c = [F(x) for x in re.findall(r"-?\d+\.\d+(?=f)", body)]
    u2 = u * u
    s = (F(1) / (F(1) + np.exp2((u * _fma(u2, b, a)).astype(np.float64)).astype(F))).astype(F)
    g = u * s
    return g, _fma(_fma(-g, s, g), _fma(u2, d, c), s)


def _tanh_library(u):
    """Likewise the scalar kernel's, with a tanh that is rounded once."""
    k0, k1 = F(0.7978845608028654), F(0.044715)
    t = np.tanh((k0 * (u + k1 * u * u * u)).astype(np.float64)).astype(F)
    h = F(0.5) * (F(1) + t)
    return u * h, h + F(0.5) * u * (F(1) - t * t) * k0 * (F(1) + F(3) * k1 * u * u)


def _tanh_exact(u):
    u = u.astype(np.float64)
    k0, k1 = math.sqrt(2 / math.pi), 0.044715
    s = 1 / (1 + np.exp(-2 * k0 * (u + k1 * u ** 3)))
    return u * s, s + 2 * u * s * (1 - s) * k0 * (1 + 3 * k1 * u * u)


def test_tanh_form_in_fp32():
    rng = np.random.default_rng(0)

    def errors(f, u):
        return [np.linalg.norm(a - b) / np.linalg.norm(b) for a, b in zip(f(u), _tanh_exact(u))]

    # a handful of roundings of 2^-24 = 6e-8 at most each; the library's form has one or two fewer, and cancels in the lower tail
    u = rng.standard_normal(1 << 18).astype(F)
    own, lib = errors(_tanh_form, u), errors(_tanh_library, u)
    assert own[0] < 6e-8 and own[1] < 9e-8 and own[0] < 1.4 * lib[0] and own[1] < 1.8 * lib[1], (own, lib)
    tail = np.linspace(-6.0, -3.0, 1 << 16).astype(F)
    own, lib = errors(_tanh_form, tail), errors(_tanh_library, tail)
    assert max(own) < 4e-7 and min(lib) > 2e-5, (own, lib)
    wide = np.linspace(-9.0, 9.0, 1 << 16).astype(F)
    value, slope = (np.abs(a - b) for a, b in zip(_tanh_form(wide), _tanh_exact(wide)))
    assert value.max() < 8e-7 and slope.max() < 3e-6, (value.max(), slope.max())
    # what is stored is rounded to bf16: the same error from float64 in both forms, to a part in ten thousand
    import torch
    exact = _tanh_exact(u)
    for i in range(2):
        both = [np.linalg.norm(torch.from_numpy(f(u)[i]).bfloat16().double().numpy() - exact[i]) / np.linalg.norm(exact[i])
                for f in (_tanh_form, _tanh_library)]
        assert abs(both[0] / both[1] - 1.0) < 1e-4, both
