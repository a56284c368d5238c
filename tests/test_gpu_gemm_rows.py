"""Tall bfloat16 A times a small B with result and mask in bfloat16, in the range of the kernel that keeps a row block in registers:
widths and reductions around its pieces, ragged rows, padded and tight leading dimensions, both forms of B, every epilogue; and just outside
of it, where the kernel for all tall products works."""
import numpy as np
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


# Products of more than 65536 rows: a workgroup has several blocks of rows, and the next one is requested while this one is multiplied and
# stored.  Beyond 160 MB of operands (and for leading dimensions that are odd, widths that are no multiple of four, and narrow results of
# rows that are a multiple of 128 bytes apart) the other kernel works.
@pytest.mark.parametrize("M,N,K,masked,rows", [
    (100003, 256, 256, False, True), (100003, 256, 256, True, True), (131099, 172, 196, False, True), (131099, 172, 196, True, True),
    (99001, 256, 172, True, True), (131099, 100, 132, True, True), (131099, 256, 172, False, True),
    (163841, 256, 256, False, False), (109227, 256, 256, True, False), (245000, 172, 172, False, False), (163000, 172, 172, True, False),
    (228000, 256, 112, False, False), (70001, 102, 130, True, False), (4100, 198, 70, False, False),
    (4097, 128, 256, False, False), (4097, 128, 256, True, False), (65536, 72, 192, False, False), (65536, 72, 192, True, True), (65537, 128, 256, True, True),
    (110001, 192, 256, False, False), (110000, 192, 256, False, True), (110001, 192, 256, True, True), (65537, 128, 256, False, False), (65537, 128, 192, False, True),
    (4097, 132, 256, False, True), (4097, 128, 128, False, True), (4097, 128, 252, False, True)])
@pytest.mark.parametrize("tb", [False, True])
def test_many_rows(M, N, K, masked, rows, tb):
    gen = torch.Generator(device=DEV).manual_seed(M + N + tb)
    A = torch.randn(M, K, generator=gen, device=DEV).bfloat16()
    B = torch.randn((N, K) if tb else (K, N), generator=gen, device=DEV)
    mask = torch.randn(M, N, generator=gen, device=DEV).bfloat16() if masked else None
    C = torch.full((M + 1, N), 7.0, device=DEV).bfloat16()
    ctx().profile(True)
    sg.sgnn_gemm(ctx(), False, tb, A, B, None, sg.SGNN_BF16_MFMA, C[:M], mask=mask)
    names = [r[0] for r in ctx().profile_read()]
    ctx().profile(False)
    assert ("gemm_rows_kernel" in names) == rows and ("gemm_skinny_bf16_kernel" in names) != rows
    Bd = B.bfloat16().double()
    ref, scale = A.double() @ (Bd.T if tb else Bd), A.double().abs() @ (Bd.T if tb else Bd).abs()
    if masked:
        ref = ref * (mask.double() > 0)
    assert torch.all((C[:M].double() - ref).abs() <= K * 2.0 ** -23 * scale + 2.0 ** -8 * ref.abs())
    assert torch.all(C[M] == 7.0)


@pytest.mark.parametrize("n,d_in,d_out", [(4100, 172, 100), (70001, 256, 256)])
def test_rows_through_an_index(n, d_in, d_out):
    # a transform-first layer on gathered rows: the product reads row idx[i] of the features, the aggregation is one entry of 1 a row
    gen = torch.Generator(device=DEV).manual_seed(n)
    H = torch.randn(n + 999, d_in, generator=gen, device=DEV).bfloat16()
    W = torch.randn(d_in, d_out, generator=gen, device=DEV)
    idx = torch.randperm(n + 999, generator=gen, device=DEV)[:n].int()
    A = sg.Csr.from_arrays(n, n, np.arange(n + 1), np.arange(n), np.ones(n, np.float32), DEV)
    Y = torch.empty((n, d_out), dtype=torch.bfloat16, device=DEV)
    ctx().profile(True)
    sg.sgnn_gcn_fwd(ctx(), A, H, W, None, sg.SGNN_BF16_MFMA | sg.SGNN_XFORM_FIRST, Y, None, row_index=idx)
    names = [r[0] for r in ctx().profile_read()]
    ctx().profile(False)
    assert "gemm_rows_kernel" in names
    G = H[idx.long()].double()
    ref, scale = G @ W.bfloat16().double(), G.abs() @ W.bfloat16().double().abs()
    # the product rounded to bfloat16 once; the aggregation copies it
    assert torch.all((Y.double() - ref).abs() <= d_in * 2.0 ** -23 * scale + 2.0 ** -8 * ref.abs())


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
