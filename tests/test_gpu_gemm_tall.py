"""The tall-operand product with both sides stored as bfloat16 and nothing beside them (csrc/gemm_tall.hip): widths and reductions at the edges
of its frames, odd ones, ragged rows, padding that holds NaN, bias and ReLU, the result in the place of the operand."""
import pytest
import torch

import paper_2604_02651_amd as sg
from gpu_util import DEV, ctx

pytestmark = pytest.mark.gpu


# more than 160 MB of operands, or a result of up to 64 columns and 100000 rows: what gemm_rows.hip does not take
SIZES = [(170001, 256, 256), (310017, 172, 100), (262177, 128, 192), (200003, 193, 255), (520001, 100, 64), (400000, 129, 65), (100000, 64, 256),
         (100033, 47, 256), (100001, 1, 129), (150007, 33, 193), (262145, 255, 57), (4096, 99, 256), (4127, 70, 1), (9999, 250, 130), (33000, 66, 65)]


@pytest.mark.parametrize("M,N,K", SIZES)
def test_against_float64(M, N, K):
    gen = torch.Generator(device=DEV).manual_seed(M + N + K)
    pad = -K % 8 + 8 * (N % 2)
    A = torch.full((M, K + pad), float("nan"), device=DEV, dtype=torch.bfloat16)
    A[:, :K] = torch.randn(M, K, generator=gen, device=DEV).bfloat16()
    B = torch.randn(K, N + N % 3, generator=gen, device=DEV)[:, :N]
    bias = torch.randn(N, generator=gen, device=DEV)
    C = torch.full((M + 1, N + -N % 8 + 8), 7.0, device=DEV).bfloat16()
    for use_bias, relu in ((False, False), (True, True)):
        C.fill_(7.0)
        ctx().profile(True)
        sg.sgnn_gemm(ctx(), False, False, A[:, :K], B, bias if use_bias else None, sg.SGNN_BF16_MFMA | (sg.SGNN_RELU if relu else 0), C[:M, :N])
        tags = [r[1] for r in ctx().profile_read()]
        ctx().profile(False)
        assert any(t.startswith("NN tall") for t in tags)
        for r0 in range(0, M, 1 << 16):
            a = A[r0:min(r0 + (1 << 16), M), :K].double()
            want, scale = a @ B.bfloat16().double(), a.abs() @ B.bfloat16().double().abs() + 8
            if use_bias:
                want = want + bias.double()
            if relu:
                want = want.clamp(min=0)
            # fp32 sums of K terms, then one rounding to bfloat16 (relative 2^-9, half an ulp of 8 bits)
            assert torch.all((C[r0:r0 + a.shape[0], :N].double() - want).abs() <= K * 2.0 ** -23 * scale + 2.0 ** -8 * want.abs())
        assert torch.all(C[M] == 7.0) and torch.all(C[:, N:] == 7.0)


def test_result_in_the_place_of_the_operand():
    M, N = 200017, 256
    gen = torch.Generator(device=DEV).manual_seed(5)
    A, B = torch.randn(M, N, generator=gen, device=DEV).bfloat16(), torch.randn(N, N, generator=gen, device=DEV)
    C = torch.empty_like(A)
    sg.sgnn_gemm(ctx(), False, False, A, B, None, sg.SGNN_BF16_MFMA, C)
    sg.sgnn_gemm(ctx(), False, False, A, B, None, sg.SGNN_BF16_MFMA, A)
    assert torch.equal(A, C)


# rows that end four columns into a chunk of eight (one store there instead of three), in every number of tiles
@pytest.mark.parametrize("M,N,K", [(33000, 68, 65), (33001, 132, 130), (12345, 100, 256), (40003, 164, 70), (250007, 36, 101), (350003, 20, 129),
                                   (33000, 252, 193)])
def test_rows_that_end_in_half_a_chunk(M, N, K):
    test_against_float64(M, N, K)


# just inside the ranges that this kernel has
@pytest.mark.parametrize("M,N,K", [(39999, 70, 101), (500003, 90, 65), (75001, 99, 170), (24999, 69, 57), (80001, 99, 30), (59999, 134, 63), (300007, 196, 17), (250001, 62, 65), (350000, 32, 256), (100000, 3, 159),
                                   (99999, 255, 17)])
def test_edges_of_its_ranges(M, N, K):
    test_against_float64(M, N, K)


# what the kernel of gemm.hip is the better one for: up to 64 columns with few rows or steps, whole tiles of few slices, few steps
@pytest.mark.parametrize("M,N,K", [(99999, 64, 256), (200001, 47, 128), (131072, 20, 172), (65537, 128, 192), (40001, 96, 250), (100001, 70, 57),
                                   (60001, 150, 64), (100003, 172, 57),
                                   (40001, 70, 65), (499999, 90, 128), (74999, 99, 129), (25000, 96, 64), (40000, 128, 1), (40003, 160, 40), (299999, 224, 64), (349999, 5, 130), (100000, 4, 160), (100000, 255, 32)])
def test_left_to_the_other_kernel(M, N, K):
    gen = torch.Generator(device=DEV).manual_seed(M + N + K)
    A = torch.randn(M, K + -K % 8, generator=gen, device=DEV).bfloat16()[:, :K]
    B, bias = torch.randn(K, N, generator=gen, device=DEV), torch.randn(N, generator=gen, device=DEV)
    C = torch.full((M + 1, N + -N % 8 + 8), 7.0, device=DEV).bfloat16()
    ctx().profile(True)
    sg.sgnn_gemm(ctx(), False, False, A, B, bias, sg.SGNN_BF16_MFMA | sg.SGNN_RELU, C[:M, :N])
    records = ctx().profile_read()
    ctx().profile(False)
    assert records and not any(r[1].startswith("NN tall") for r in records)
    a, b = A.double(), B.bfloat16().double()
    want = (a @ b + bias.double()).clamp(min=0)
    assert torch.all((C[:M, :N].double() - want).abs() <= K * 2.0 ** -23 * (a.abs() @ b.abs() + 8) + 2.0 ** -8 * want.abs())
    assert torch.all(C[M] == 7.0) and torch.all(C[:, N:] == 7.0)
