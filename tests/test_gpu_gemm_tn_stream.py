"""Streaming weight gradient (both operands bfloat16): every frame width, ragged reductions, padding that holds NaN, against
the same product of the stored values in 64 bits."""
import pytest
import torch

import paper_2604_02651_amd as sg
from gpu_util import DEV, ctx

pytestmark = pytest.mark.gpu


def _operand(K, M, seed, pad):
    """K x M view of a matrix whose padding columns hold NaN."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    m = torch.full((K, (M + 7) // 8 * 8 + pad), float("nan"), dtype=torch.bfloat16, device=DEV)
    m[:, :M] = torch.randn((K, M), device=DEV, generator=gen)
    return m[:, :M]


@pytest.mark.parametrize("K", [8191, 8192, 8193, 8223, 8255, 40003])
@pytest.mark.parametrize("M,N", [(256, 256), (255, 65), (129, 7), (128, 129), (100, 128), (65, 1), (64, 255), (33, 66), (3, 64), (1, 1)])
def test_against_64_bits(M, N, K):
    A, B = _operand(K, M, 1, 0), _operand(K, N, 2, 8 * (K % 3))
    ctx().reserve(1 << 16, 1 << 16, 1 << 16, 256, 1 << 16)
    C, cs = torch.full((M, N + 1), 7.0, device=DEV), torch.empty(N, device=DEV)
    sg.sgnn_gemm(ctx(), True, False, A, B, None, sg.SGNN_BF16_MFMA, C[:, :N], b_colsum=cs)
    # the products are exact in fp32: sums of K of them in at most 256 ranges; 2^-21 of the sum of magnitudes covers their rounding
    A64, B64 = A.double(), B.double()
    assert torch.all((C[:, :N].double() - A64.T @ B64).abs() <= (A64.abs().T @ B64.abs()) * 2.0 ** -21)
    assert torch.all((cs.double() - B64.sum(0)).abs() <= B64.abs().sum(0) * 2.0 ** -21)
    assert torch.all(C[:, N] == 7.0)
    C2 = torch.empty((M, N), device=DEV)
    sg.sgnn_gemm(ctx(), True, False, A, B, None, sg.SGNN_BF16_MFMA, C2)
    assert torch.equal(C2, C[:, :N])


def test_infinite_last_row():
    # the rows that fill up the last slice repeat the last one and must not reach the sums
    K, M, N = 8201, 70, 40
    A, B = _operand(K, M, 1, 0), _operand(K, N, 2, 0)
    A[K - 1, 3] = float("inf")
    B[K - 1] = 1.0
    C = torch.empty((M, N), device=DEV)
    sg.sgnn_gemm(ctx(), True, False, A, B, None, sg.SGNN_BF16_MFMA, C)
    assert torch.all(torch.isinf(C[3])) and torch.all(torch.isfinite(C[:3])) and torch.all(torch.isfinite(C[4:]))
