"""Tall bfloat16 A times a small B with result and mask in bfloat16, in the range of the kernel that keeps a row block in registers:
widths and reductions around its pieces, ragged rows, padded and tight leading dimensions, both forms of B, every epilogue."""
import pytest
import torch

import paper_2604_02651_amd as sg
from gpu_util import DEV, ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(4096, 256, 256), (4097, 68, 8), (5001, 128, 64), (4127, 132, 68), (4128, 172, 256), (70001, 192, 100),
                                   (4352, 196, 132), (9999, 200, 20), (4100, 252, 192), (4100, 256, 196), (66000, 256, 12), (4096, 72, 252)])
@pytest.mark.parametrize("tb", [False, True])
def test_against_float64(M, N, K, tb):
    gen = torch.Generator().manual_seed(M + N)
    pad_a, pad_c = 4 * (N % 3), 4 * (K % 2) + 2 * (M % 2)
    A = torch.randn(M, K + pad_a, generator=gen).to(DEV).bfloat16()[:, :K]
    B = torch.randn((N, K) if tb else (K, N), generator=gen).to(DEV)
    bias = torch.randn(N, generator=gen).to(DEV)
    mask = torch.randn(M, N + 4, generator=gen).to(DEV).bfloat16()[:, :N]
    mask[:, ::7] = 0
    ref = A.double() @ (B.bfloat16().double().T if tb else B.bfloat16().double())
    scale = A.double().abs() @ (B.bfloat16().double().abs().T if tb else B.bfloat16().double().abs())

    def check(got, want):
        # fp32 sums of K terms, then one rounding to bfloat16 (relative 2^-9, half an ulp of 8 bits)
        assert torch.all((got.double() - want).abs() <= K * 2.0 ** -23 * (scale + 8) + 2.0 ** -8 * want.abs())

    for use_bias, relu, masked in ((False, False, False), (True, False, False), (True, True, False), (False, False, True)):
        C = torch.full((M + 1, N + pad_c), 7.0, device=DEV).bfloat16()
        sg.sgnn_gemm(ctx(), False, tb, A, B, bias if use_bias else None, sg.SGNN_BF16_MFMA | (sg.SGNN_RELU if relu else 0), C[:M, :N],
                     mask=mask if masked else None)
        want = ref + bias.double() if use_bias else ref
        if relu:
            want = want.clamp(min=0)
        if masked:
            want = want * (mask.double() > 0)
        check(C[:M, :N], want)
        assert torch.all(C[M] == 7.0) and torch.all(C[:, N:] == 7.0)


@pytest.mark.parametrize("M,N,K", [(4097, 128, 128), (4128, 256, 256), (4321, 172, 172), (66000, 72, 72)])
def test_result_in_the_place_of_an_operand(M, N, K):
    # every row is read by the wavefront that writes it and by no other, the last one too (M % 256 from 1 to 224: wavefronts without rows)
    gen = torch.Generator().manual_seed(M)
    A = torch.randn(M, K, generator=gen).to(DEV).bfloat16()
    B = torch.randn(K, N, generator=gen).to(DEV)
    mask = torch.randn(M, N, generator=gen).to(DEV).bfloat16()
    ref, scale = A.double() @ B.bfloat16().double(), A.double().abs() @ B.bfloat16().double().abs()
    masked = ref * (mask.double() > 0)
    for _ in range(4):
        C = mask.clone()
        sg.sgnn_gemm(ctx(), False, False, A, B, None, sg.SGNN_BF16_MFMA, C, mask=C)
        assert torch.all((C.double() - masked).abs() <= K * 2.0 ** -23 * scale + 2.0 ** -8 * masked.abs())
        C = A.clone()
        sg.sgnn_gemm(ctx(), False, False, C, B, None, sg.SGNN_BF16_MFMA, C)
        assert torch.all((C.double() - ref).abs() <= K * 2.0 ** -23 * scale + 2.0 ** -8 * ref.abs())


def test_infinities_beyond_the_reduction_do_not_count():
    # the last 16 bytes of a row of A reach over the end of a piece: what is there is not multiplied with zeros
    M, N, K = 4099, 100, 68
    A = torch.full((M, 80), float("inf"), device=DEV).bfloat16()
    A[:, :K] = torch.randn(M, K, generator=torch.Generator().manual_seed(3)).to(DEV).bfloat16()
    B = torch.ones(K, N, device=DEV)
    C = torch.empty((M, N), device=DEV, dtype=torch.bfloat16)
    sg.sgnn_gemm(ctx(), False, False, A[:, :K], B, None, sg.SGNN_BF16_MFMA, C)
    want = A[:, :K].double().sum(1, keepdim=True).expand(M, N)
    assert torch.all((C.double() - want).abs() <= K * 2.0 ** -23 * A[:, :K].double().abs().sum(1, keepdim=True) + 2.0 ** -8 * want.abs())
