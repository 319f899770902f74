"""Kernels for sizes that no tile divides, at the sizes where they can go wrong: one less, exactly and one more than a
tile, single rows, contractions that end inside a slab.  Against float64 products of the same rounded operands."""
import numpy as np
import pytest
import torch

import paper_2204_06514_amd as fax
from helpers import DEV, TDTYPE, CODE, to_dev, to_np, rel_max, rel_fro
from workloads import round_to_bf16

pytestmark = pytest.mark.gpu

# M, N, K.  The masked-edge GEMM keeps what is contiguous in memory a multiple of 8 elements; the rest is free.
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
