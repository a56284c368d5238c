"""Sums of the partial products of a split reduction (csrc/gemm_reduce.hip) through weight gradients: at most 16 of them, up to 32 of at least 65536
elements (an element a thread) and the others (eight wavefronts an element), with the column sums next to them and without."""
import pytest
import torch

import paper_2604_02651_amd as sg
from gpu_util import DEV, ctx

pytestmark = pytest.mark.gpu


# rows x columns of the result, reduction, bfloat16: 16, 24, 32 and more partial products on both sides of 65536 elements; ragged ends of the blocks
@pytest.mark.parametrize("M,N,K,bf16,few", [
    (16, 16, 4096, False, True), (608, 256, 4096, True, True), (400, 404, 16384, True, True), (300, 300, 12000, True, True), (256, 256, 4096, False, True),
    (256, 260, 4097, False, True), (256, 256, 4224, False, False), (252, 256, 4096, False, False), (100, 64, 6000, True, False), (4, 8, 8192, False, False),
    (255, 257, 30011, False, False)])
def test_weight_gradient_and_column_sums(M, N, K, bf16, few):
    gen = torch.Generator(device=DEV).manual_seed(M + N + K)
    dtype = torch.bfloat16 if bf16 else torch.float32
    A, B = (torch.randn((K, d), generator=gen, device=DEV).to(dtype) for d in (M, N))
    frame, db = torch.full((M + 1, N), 9.0, device=DEV), torch.full((N,), 9.0, device=DEV)
    ctx().reserve(1 << 20, 1 << 20, 65536, 640, 1 << 20)
    first = None
    for with_db in (True, False, True):
        ctx().profile(True)
        sg.sgnn_gemm(ctx(), True, False, A, B, None, sg.SGNN_BF16_MFMA if bf16 else 0, frame[:M], b_colsum=db if with_db else None)
        tags = [r[1] for r in ctx().profile_read() if r[0] == "splitk_reduce_kernel"]
        ctx().profile(False)
        assert len(tags) == 1 and ("few" in tags[0]) == few
        ref, scale = A.double().T @ B.double(), A.double().abs().T @ B.double().abs()
        # fp32 sums in chains of up to a few hundred terms of random sign: 16 units of 2^-24 of the sum of magnitudes
        assert torch.all((frame[:M].double() - ref).abs() <= 2.0 ** -20 * scale) and torch.all(frame[M] == 9.0)
        assert torch.all((db.double() - B.double().sum(0)).abs() <= 2.0 ** -20 * B.double().abs().sum(0))
        first = frame.clone() if first is None else first
        assert torch.equal(frame, first)
