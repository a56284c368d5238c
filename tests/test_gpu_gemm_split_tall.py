"""Split fp32 products of a tall A and a small B (csrc/gemm_split_tall.hip), which take over where the tiles of gemm_split.hip are more than the
compute units: widths and reductions at the edges of the frames and pieces, ragged rows, operands with odd leading dimensions and one
element behind a 16-byte boundary, bias and ReLU, and the values for which the split does not hold."""
import pytest
import torch

import paper_2604_02651_amd as sg
from gpu_util import DEV, ctx

pytestmark = pytest.mark.gpu

# (M, N, K): frames of 128 / 192 / 256 steps and of 128 / 256 columns, slices of 64 and 32 rows
SIZES = [(33000, 256, 256), (32769, 129, 65), (40001, 255, 193), (17000, 200, 200), (36007, 130, 128), (65537, 128, 256), (66001, 65, 67),
         (70003, 97, 131), (33001, 66, 192), (34000, 254, 254)]


def operand(rows, cols, seed, pad=3, offset=1):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    flat = torch.randn(rows * (cols + pad) + offset, device=DEV, generator=gen)
    return flat[offset:].view(rows, cols + pad)[:, :cols]


def product(A, B, tb, bias=None, relu=False, pad=2):
    M, N = A.shape[0], B.shape[0] if tb else B.shape[1]
    out = torch.full((M + 1, N + pad), 9.0, device=DEV)
    ctx().profile(True)
    sg.sgnn_gemm(ctx(), False, tb, A, B, bias, sg.SGNN_RELU if relu else 0, out[:M, :N])
    tags = [r[1] for r in ctx().profile_read()]
    ctx().profile(False)
    assert len(tags) == 1 and " tall " in tags[0]
    assert torch.all(out[M] == 9.0) and torch.all(out[:, N:] == 9.0)
    return out[:M, :N]


@pytest.mark.parametrize("tb", [False, True])
@pytest.mark.parametrize("M,N,K", SIZES)
def test_against_float64(M, N, K, tb):
    A, B = operand(M, K, 1), operand(N, K, 2) if tb else operand(K, N, 2)
    bias = operand(1, N, 3)[0].contiguous()
    A64, B64 = A.double(), B.double().T if tb else B.double()
    ref, scale = A64 @ B64, A64.abs() @ B64.abs()
    C = product(A, B, tb)
    # 24-bit operands, fp32 accumulation in a few dozen steps of random sign
    assert torch.all((C.double() - ref).abs() <= scale * 2.0 ** -22)
    assert (C.double() - ref).norm() <= 2e-7 * ref.norm()
    assert torch.equal(product(A, B, tb, bias, True), (C + bias).relu())


@pytest.mark.parametrize("tb", [False, True])
def test_same_sums_as_the_tiles(tb):
    # the first rows alone are a call of gemm_split.hip: the same products in the same order
    A, B = operand(33000, 256, 1), operand(256, 256, 2)
    few = torch.empty((5000, 256), device=DEV)
    sg.sgnn_gemm(ctx(), False, tb, A[:5000], B, None, 0, few)
    assert torch.equal(product(A, B, tb)[:5000], few)


@pytest.mark.parametrize("tb", [False, True])
def test_values_the_split_does_not_hold_for(tb):
    M, N, K = 33003, 140, 90
    A, B = operand(M, K, 1).contiguous(), operand(K, N, 2).contiguous()

    def mul(A, B):
        return product(A, B.T.contiguous() if tb else B, tb).double()
    plain = mul(A, B)
    # tiny values in one slice, and in the first and the last row: the other slices keep their bits
    T = A.clone()
    for row in (0, 32000, M - 1):
        T[row] *= 2.0 ** -120
    got, ref = mul(T, B), T.double() @ B.double()
    for row in (0, 32000, M - 1):
        assert (got[row] - ref[row]).norm() <= 1e-6 * ref[row].norm()
    assert torch.equal(got[64:31900], plain[64:31900])
    for e in (-120, -149):          # all of B
        Bs = (B * 2.0 ** e) if e > -140 else torch.full_like(B, 2.0 ** e)
        As = A * 2.0 ** 30
        ref = As.double() @ Bs.double()
        assert (mul(As, Bs) - ref).norm() <= 1e-6 * ref.norm()
    A[3, 5], A[20077, 0], B[7, 100] = float("inf"), float("nan"), -float("inf")
    A[140, 2] = 3.4e38                  # finite, but rounds up to infinity in bfloat16
    B[2] = B[2].clamp(-0.4, 0.4)
    ref, got = A.double() @ B.double(), mul(A, B)
    assert torch.equal(torch.isnan(got), torch.isnan(ref)) and torch.equal(torch.isinf(got), torch.isinf(ref))
    fine = torch.isfinite(ref)
    assert torch.equal(got[torch.isinf(ref)], ref[torch.isinf(ref)])
    assert (got[fine] - ref[fine]).norm() <= 1e-6 * ref[fine].norm()


# B given N x K with K no multiple of 64: the ends of its rows; just above one tile a compute unit
@pytest.mark.parametrize("tb", [False, True])
@pytest.mark.parametrize("M,N,K", [(16500, 256, 96), (33000, 128, 200), (33000, 96, 68)])
def test_ends_of_the_rows_of_b(M, N, K, tb):
    test_against_float64(M, N, K, tb)
