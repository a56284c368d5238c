"""The kernel that computes both products of a layer's backward pass from one read of their operands (bfloat16 storage, csrc/gemm_bwd.hip),
reached through sgnn_gcn_bwd with the identity as the sparse matrix: aggregate first dW = T^T dY, db, dH = dY W^T; transform first
dW = H^T dY, dH = (dY W^T) where H > 0.  Reference: the same products in float64 on the CPU."""
import numpy as np
import pytest
import torch

import paper_2604_02651_amd as sg
from gpu_util import DEV, ctx

pytestmark = pytest.mark.gpu


def identity(n):
    return sg.Csr.from_arrays(n, n, np.arange(n + 1), np.arange(n), np.ones(n, np.float32), DEV)


def stored(x, pad):
    """x as bfloat16 with `pad` more columns that hold NaN."""
    m = torch.full((x.shape[0], x.shape[1] + pad), float("nan"), dtype=torch.bfloat16)
    m[:, :x.shape[1]] = x
    return m.to(DEV)[:, :x.shape[1]]


def pad8(d):
    return (-d) % 8 + 8


# widths at the edges of the frames (64 / 128 / 192 / 256 columns), rows at the edges of slices and of a workgroup's share of them
SIZES = [(8192, 256, 256), (8193, 256, 255), (10007, 256, 193), (16415, 248, 192), (9999, 136, 129), (8230, 256, 128), (8221, 200, 47), (12345, 129, 1),
         (8192, 128, 256), (8255, 72, 200), (30011, 65, 128), (8197, 104, 65), (9001, 128, 30), (70001, 256, 256), (110016, 128, 256),
         (110001, 96, 190), (110049, 128, 66)]


@pytest.mark.parametrize("K,M,N", SIZES)
@pytest.mark.parametrize("xform", [False, True])
def test_both_products(K, M, N, xform):
    gen = torch.Generator().manual_seed(K + M + N)
    X = torch.randn((K, M), generator=gen).relu_().to(torch.bfloat16)
    D = torch.randn((K, N), generator=gen).to(torch.bfloat16)
    W = torch.randn((M, N), generator=gen) / N ** 0.5
    A, Xd, Dd, Wd = identity(K), stored(X, pad8(M)), stored(D, pad8(N)), W.to(DEV)
    ctx().reserve(K, K, K, 256, K)
    flags = sg.SGNN_BF16_MFMA | (sg.SGNN_XFORM_FIRST if xform else 0)

    def call(dH):
        dW, db = torch.full((M, N), float("nan"), device=DEV), torch.full((N,), float("nan"), device=DEV)
        sg.sgnn_gcn_bwd(ctx(), A, Xd, Wd, None, Dd, flags, dH, dW, None if xform else db, H_in=Xd if xform else None)
        return dW, db

    frame = torch.full((K, M + pad8(M)), 7.0, dtype=torch.bfloat16, device=DEV)
    dH = frame[:, :M]
    dW, db = call(dH)
    X64, D64, W64 = X.double(), D.double(), W.to(torch.bfloat16).double()
    # fp32 sums of K terms in 32-row slices: far below the 1e-4 that the weight gradients are held to elsewhere
    ref = X64.T @ D64
    assert (dW.cpu().double() - ref).norm() / ref.norm() < 1e-5
    if not xform:
        assert (db.cpu().double() - D64.sum(0)).abs().max() < 1e-5 * D64.abs().sum(0).max()
    ref = D64 @ W64.T
    if xform:
        ref = torch.where(X > 0, ref, 0.0)
    # one rounding to bfloat16 (half an ulp, 2^-9) behind fp32 sums
    bound = ref.abs() * 2.0 ** -8 + 1e-5 * (D64.abs() @ W64.abs().T)
    assert ((dH.cpu().double() - ref).abs() <= bound).all()
    assert (frame[:, M:] == 7.0).all()
    again = torch.zeros_like(dH)
    dW2, db2 = call(again)
    assert torch.equal(dW, dW2) and torch.equal(dH, again) and (xform or torch.equal(db, db2))
    if xform:          # the gradient in the place of the layer's input
        dW3, _ = call(Xd)
        assert torch.equal(dW3, dW) and torch.equal(Xd, dH)


def test_infinities_stay_in_their_rows():
    K, M, N = 8200, 136, 70
    gen = torch.Generator().manual_seed(1)
    X = torch.randn((K, M), generator=gen).to(torch.bfloat16)
    D = torch.randn((K, N), generator=gen).to(torch.bfloat16)
    D[8199, 69] = float("inf")
    W = torch.rand((M, N), generator=gen) + 0.5
    dH, dW, db = stored(torch.zeros(K, M), 8), torch.zeros((M, N), device=DEV), torch.zeros(N, device=DEV)
    sg.sgnn_gcn_bwd(ctx(), identity(K), stored(X, 8), W.to(DEV), None, stored(D, 10), sg.SGNN_BF16_MFMA, dH, dW, db)
    assert torch.isfinite(dH[:8199]).all() and (dH[8199] == float("inf")).all()
    assert torch.isfinite(dW[:, :69]).all() and torch.isinf(dW[:, 69]).all()
    assert torch.isfinite(db[:69]).all() and db[69] == float("inf")


def backward_kernels(call):
    ctx().profile(True)
    call()
    tags = [r[1] for r in ctx().profile_read() if r[0] == "gemm_bwd_kernel"]
    ctx().profile(False)
    return tags


# The results of the two separate products meet the same bounds: that the kernel is the one that ran.  Narrow X beside wide D has it from
# 110000 rows on; transform first, M is a multiple of eight (the columns behind dH are the caller's)
@pytest.mark.parametrize("K,M,N,xform", [
    (8192, 256, 256, False), (8192, 256, 256, True), (8193, 256, 255, True), (10007, 256, 193, False), (16415, 248, 192, True), (9999, 136, 129, False),
    (12345, 129, 1, False), (8221, 200, 47, True), (9001, 128, 30, False), (8200, 72, 64, True), (8201, 65, 33, False), (110003, 65, 128, False),
    (110011, 72, 200, False), (110011, 72, 200, True), (110005, 104, 65, False), (110005, 104, 65, True), (110001, 96, 190, True), (110016, 128, 256, False),
    (16000, 192, 250, False), (9003, 160, 224, True), (9003, 136, 192, False), (8205, 256, 96, False), (8195, 256, 3, True), (8200, 256, 4, False)])
def test_one_pass_for_both(K, M, N, xform):
    tags = backward_kernels(lambda: test_both_products(K, M, N, xform))
    assert len(tags) == 1 and tags[0].startswith("bwd %dx%dx%d " % (M, N, K)) and ("mask" in tags[0]) == xform


@pytest.mark.parametrize("K,M,N,xform", [
    (8191, 256, 256, False), (12345, 64, 64, False), (8192, 128, 256, False), (8255, 72, 200, True), (109999, 65, 128, False), (12345, 129, 1, True),
    (15999, 192, 193, False)])
def test_two_products_where_it_does_not_pay_or_fit(K, M, N, xform):
    assert not backward_kernels(lambda: test_both_products(K, M, N, xform))


def test_infinities_in_the_one_pass():
    assert backward_kernels(test_infinities_stay_in_their_rows)
