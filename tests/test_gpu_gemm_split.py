"""fp32 products whose operands are split into bfloat16 parts: tile edges, reduction tails, every layout and epilogue, unaligned
operands, gathered rows, short and split reductions, and the values for which the split does not hold."""
import numpy as np
import pytest
import torch

import paper_2604_02651_amd as sg
from gpu_util import DEV, TOL_F32, ctx, rel_err

pytestmark = pytest.mark.gpu

# (M, N, K): each tile shape with remainders of 1 to 3 rows, columns and reduction steps
SHAPES = [(4, 4, 4), (5, 7, 6), (63, 33, 35), (64, 64, 64), (65, 66, 67), (129, 65, 47), (1057, 200, 200), (130, 257, 1001),
          (16900, 65, 70), (20483, 130, 33), (40963, 129, 101), (41000, 200, 32)]
TN_SHAPES = [(4, 4, 4), (5, 33, 9), (64, 34, 255), (53, 200, 1057), (100, 64, 3001), (47, 100, 9001), (130, 66, 8200), (257, 131, 8195),
             (608, 256, 8192), (65, 129, 30011)]


def _operand(rows, cols, seed, pad=3, offset=1, scale=1.0):
    """rows x cols view with an odd leading dimension, one element behind a 16-byte boundary."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    flat = torch.randn(rows * (cols + pad) + offset, device=DEV, generator=gen) * scale
    return flat[offset:].view(rows, cols + pad)[:, :cols]


def _check(got, A64, B64, ref):
    """Within 2^-22 of the sum of the products' magnitudes, entry by entry: 24-bit operands, fp32 accumulation in at most a few
    hundred steps of random sign; and 1e-6 in the 2-norm."""
    bound = (A64.abs() @ B64.abs()) * 2.0 ** -22 + 1e-30
    assert torch.all((got.double() - ref).abs() <= bound)
    assert (got.double() - ref).norm() <= 1e-6 * (A64 @ B64).norm() + 1e-30


@pytest.mark.parametrize("tb", [False, True])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_transform_and_input_gradient(M, N, K, tb):
    ctx().reserve(1 << 20, 1 << 20, 65536, 640, 1 << 20)
    A, B = _operand(M, K, 1), _operand(N, K, 2) if tb else _operand(K, N, 2)
    bias, mask = _operand(1, N, 3)[0].contiguous(), _operand(M, N, 4)
    A64, B64 = A.double(), B.double().T if tb else B.double()
    out = torch.full((M + 1, N + 2), 9.0, device=DEV)
    C = out[:M, :N]
    sg.sgnn_gemm(ctx(), False, tb, A, B, None, 0, C)
    _check(C, A64, B64, A64 @ B64)
    assert torch.all(out[M] == 9.0) and torch.all(out[:, N:] == 9.0)
    C2 = torch.empty((M, N), device=DEV)
    sg.sgnn_gemm(ctx(), False, tb, A, B, bias, sg.SGNN_RELU, C2, mask=mask)
    assert torch.equal(C2, (C + bias).relu() * (mask > 0))


@pytest.mark.parametrize("M,N,K", TN_SHAPES)
def test_weight_gradient_with_column_sums(M, N, K):
    ctx().reserve(1 << 20, 1 << 20, 65536, 640, 1 << 20)
    A, B = _operand(K, M, 5), _operand(K, N, 6)
    C, cs = torch.full((M, N), 9.0, device=DEV), torch.empty(N, device=DEV)
    sg.sgnn_gemm(ctx(), True, False, A, B, None, 0, C, b_colsum=cs)
    _check(C, A.double().T, B.double(), A.double().T @ B.double())
    assert rel_err(cs.cpu().numpy(), B.double().sum(0).cpu().numpy()) < TOL_F32
    again, cs2 = torch.empty_like(C), torch.empty_like(cs)
    sg.sgnn_gemm(ctx(), True, False, A, B, None, 0, again, b_colsum=cs2)
    assert torch.equal(again, C) and torch.equal(cs2, cs)                    # bit-reproducible


@pytest.mark.parametrize("M,N,K,tile", [(33025, 129, 70, "256x128"), (20000, 200, 300, "256x128"), (2040, 1930, 35, "128x128"), (21001, 65, 33, "128x128"), (36000, 64, 65, "128x64"),
                                        (300, 200, 5003, "128x64"), (65, 66, 4097, "128x64"), (40, 256, 9001, "64x64")])
def test_weight_gradient_tiles(M, N, K, tile):
    # short reductions onto many tiles, middling ones onto few, results of up to 64 rows
    ctx().reserve(1 << 20, 1 << 20, 65536, 640, 1 << 20)
    A, B = _operand(K, M, 5), _operand(K, N, 6)
    C, cs = torch.full((M + 1, N + 2), 9.0, device=DEV), torch.empty(N, device=DEV)
    ctx().profile(True)
    sg.sgnn_gemm(ctx(), True, False, A, B, None, 0, C[:M, :N], b_colsum=cs)
    kernels = ctx().profile_read()
    ctx().profile(False)
    assert kernels[0][1].split()[1] == tile and (len(kernels) == 2) == (M < 2000)          # ranges for the small results only
    _check(C[:M, :N], A.double().T, B.double(), A.double().T @ B.double())
    assert rel_err(cs.cpu().numpy(), B.double().sum(0).cpu().numpy()) < TOL_F32
    assert torch.all(C[M] == 9.0) and torch.all(C[:, N:] == 9.0)


def test_column_sums_over_many_ranges():
    # 128 ranges of 256 steps, each with one and the same sum: added one after the other they are off by 32 units of 2^-24, because
    # the roundings go the same way for long.  Eight chains of 16 and three sums of those: at most 18 roundings of half a unit
    p = 1.0499153137207031
    A, B = _operand(32768, 256, 5), torch.zeros((32768, 256), device=DEV)
    B[::256] = p
    C, cs = torch.empty((256, 256), device=DEV), torch.empty(256, device=DEV)
    ctx().reserve(1 << 20, 1 << 20, 65536, 640, 1 << 20)
    sg.sgnn_gemm(ctx(), True, False, A, B, None, 0, C, b_colsum=cs)
    assert torch.all((cs.double() - 128 * p).abs() <= 18 * 2.0 ** -24 * 128 * p)


def test_short_reduction_without_scratch():
    # a reduction below 4096 steps needs none: it is then not split
    small = sg.Context(0)
    A, B = _operand(1500, 70, 5), _operand(1500, 66, 6)
    C = torch.empty((70, 66), device=DEV)
    sg.sgnn_gemm(small, True, False, A, B, None, 0, C)
    _check(C, A.double().T, B.double(), A.double().T @ B.double())
    small.close()


@pytest.mark.parametrize("tb", [False, True])
@pytest.mark.parametrize("M,N,K", [(256, 256, 65536), (257, 129, 4097), (1024, 256, 8416), (1000, 66, 5003), (300, 64, 9001), (128, 200, 4099),
                                   (64, 64, 60000), (33, 40, 8195), (5000, 200, 4160)])
def test_long_reductions_onto_few_tiles(M, N, K, tb):
    ctx().reserve(1 << 20, 1 << 20, 65536, 640, 1 << 20)
    A, B = _operand(M, K, 1), _operand(N, K, 2) if tb else _operand(K, N, 2)
    C, again = torch.full((M + 1, N + 2), 9.0, device=DEV), torch.empty((M, N), device=DEV)
    ctx().profile(True)
    sg.sgnn_gemm(ctx(), False, tb, A, B, None, 0, C[:M, :N])
    kernels = [k[0] for k in ctx().profile_read()]
    ctx().profile(False)
    assert kernels == ["gemm_split_kernel", "splitk_reduce_kernel"]          # one workgroup would walk all of K otherwise
    B64 = B.double().T if tb else B.double()
    _check(C[:M, :N], A.double(), B64, A.double() @ B64)
    assert torch.all(C[M] == 9.0) and torch.all(C[:, N:] == 9.0)
    sg.sgnn_gemm(ctx(), False, tb, A, B, None, 0, again)
    assert torch.equal(again, C[:M, :N])
    if K <= 5003:                # without scratch it is not split: one chain of K / 16 sums, to which the bounds of _check() still apply
        none = sg.Context(0)
        sg.sgnn_gemm(none, False, tb, A, B, None, 0, again)
        _check(again, A.double(), B64, A.double() @ B64)
        none.close()


def _context(scratch_bytes):
    """A context whose scratch is that and less than 1 MB more (reserve() takes 1 KB for every square of the width)."""
    c = sg.Context(0)
    c.reserve(1, 1, 1, max(1, int((scratch_bytes / 1024) ** 0.5)))
    return c


def _tn(c, A, B):
    C = torch.empty((A.shape[1], B.shape[1]), device=DEV)
    sg.sgnn_gemm(c, True, False, A, B, None, 0, C)
    return C


def test_scratch_limits():
    big = _context(1 << 28)
    # 256 tiles of 128 x 128 fill the chip without ranges, and 169 need two of them (20.5 MB): neither call needs more scratch
    for n, scratch in ((2048, 0), (1600, 22 << 20)):
        A, B = _operand(8192, n, 5), _operand(8192, n, 6)
        c = _context(scratch)
        _check(_tn(c, A, B), A.double().T, B.double(), A.double().T @ B.double())
        c.close()
    # 4096 steps and more onto few tiles are refused without scratch
    A, B = _operand(8192, 256, 5), _operand(8192, 256, 6)
    c = _context(0)
    with pytest.raises(sg.SgnnError):
        _tn(c, A, B)
    c.close()
    # the order of the sums does not follow the scratch: the same bits in every context that holds the ranges (300 x 300 x 3000:
    # 8.3 MB), and those of a single range in every context that does not
    for n, K, ample, scarce in ((300, 3000, 9 << 20, (0, 1 << 20, 4 << 20)), (257, 8195, 40 << 20, ())):
        A, B = _operand(K, n, 5), _operand(K, n, 6)
        c = _context(ample)
        assert torch.equal(_tn(c, A, B), _tn(big, A, B))
        c.close()
        single = None
        for scratch in scarce:
            c = _context(scratch)
            got = _tn(c, A, B)
            single = got if single is None else single
            assert torch.equal(got, single)
            c.close()
    big.close()


@pytest.mark.parametrize("trans", ["NN", "NT", "TN"])
def test_long_leading_dimensions(trans):
    # rows of a tile that lie more than 2^31 elements apart (features kept feature-major on a graph of tens of millions of
    # vertices): 63 steps of 35 M between the rows of a tile, 31 of 70 M between the reduction steps of a slice
    ta, tb = trans[0] == "T", trans[1] == "T"
    M, N, K, ld = 64, 60, 32, 35_000_000
    flat = torch.empty(64 * ld, device=DEV)
    narrow, wide = flat.view(64, ld), flat.view(32, 2 * ld)
    A = wide[:, :M] if ta else narrow[:, :K]
    B = narrow[:N, 1000:1000 + K] if tb else wide[:, 1000:1000 + N]
    gen = torch.Generator(device=DEV).manual_seed(8)
    for t in (A, B):
        t.copy_(torch.randn(t.shape, device=DEV, generator=gen))
    C = torch.empty((M, N), device=DEV)
    sg.sgnn_gemm(ctx(), ta, tb, A, B, None, 0, C)
    A64, B64 = (A.T if ta else A).double(), (B.T if tb else B).double()
    _check(C, A64, B64, A64 @ B64)
    del flat, narrow, wide, A, B
    torch.cuda.empty_cache()


@pytest.mark.parametrize("B,d_in,d_out", [(1500, 130, 65), (9000, 602, 70)])
def test_gathered_rows(B, d_in, d_out):
    # an input layer reads its rows through the sample: X[S] W forward, X[S]^T dP backward
    ctx().reserve(2 * B, 1 << 16, B, 640, 1 << 16)
    X, W = _operand(2 * B, d_in, 1), _operand(d_in, d_out, 2)
    S = torch.randperm(2 * B, generator=torch.Generator().manual_seed(3))[:B].sort()[0].to(torch.int32).to(DEV)
    eye = sg.Csr.from_arrays(B, B, np.arange(B + 1), np.arange(B), np.ones(B, np.float32), DEV)
    Y = torch.empty((B, d_out), device=DEV)
    sg.sgnn_gcn_fwd(ctx(), eye, X, W.contiguous(), None, sg.SGNN_XFORM_FIRST, Y, None, row_index=S)
    XS = X[S.long()].double()
    _check(Y, XS, W.double(), XS @ W.double())
    dY, dW = _operand(B, d_out, 4), torch.empty((d_in, d_out), device=DEV)
    sg.sgnn_gcn_bwd(ctx(), eye, X, W.contiguous(), None, dY, sg.SGNN_XFORM_FIRST, None, dW, None, row_index=S)
    _check(dW, XS.T, dY.double(), XS.T @ dY.double())


@pytest.mark.parametrize("trans", ["NN", "NT", "TN"])
def test_values_the_split_does_not_hold_for(trans):
    ta, tb = trans[0] == "T", trans[1] == "T"
    M, N, K = 150, 140, 90
    ctx().reserve(1 << 20, 1 << 20, 65536, 640, 1 << 20)

    def product(A, B):
        C = torch.empty((M, N), device=DEV)
        sg.sgnn_gemm(ctx(), ta, tb, A.T.contiguous() if ta else A, B.T.contiguous() if tb else B, None, 0, C)
        return C
    A, B = _operand(M, K, 1).contiguous(), _operand(K, N, 2).contiguous()
    for ea, eb in ((-116, 0), (-124, 30), (0, -120), (-70, -60), (60, 60)):     # parts below the bfloat16 range; products near it
        As, Bs = A * 2.0 ** ea, B * 2.0 ** eb
        ref = As.double() @ Bs.double()
        got = product(As, Bs)
        assert (got.double() - ref).norm() <= 1e-6 * ref.norm() + 2.0 ** -149 * K, (ea, eb)
    # every value of one operand so small that its first part is zero (up to 2^-134), down to the smallest number there is
    for e in (-136, -149):
        small = torch.full_like(A, 2.0 ** e) * torch.where(A > 0, 1.0, -1.0)
        for As, Bs in ((small, B * 2.0 ** 30), (torch.full_like(A, 2.0 ** 30), torch.full_like(B, 2.0 ** e))):
            ref = As.double() @ Bs.double()
            assert (product(As, Bs).double() - ref).norm() <= 1e-6 * ref.norm() and ref.norm() > 0, e
    A[3, 5], A[77, 0], B[7, 100] = float("inf"), float("nan"), -float("inf")
    A[140, 2] = 3.4e38                  # finite, but rounds up to infinity in bfloat16
    B[2] = B[2].clamp(-0.4, 0.4)
    ref, got = A.double() @ B.double(), product(A, B).double()
    assert torch.equal(torch.isnan(got), torch.isnan(ref)) and torch.equal(torch.isinf(got), torch.isinf(ref))
    fine = torch.isfinite(ref)
    assert torch.equal(got[torch.isinf(ref)], ref[torch.isinf(ref)])
    assert (got[fine] - ref[fine]).norm() <= 1e-6 * ref[fine].norm()
