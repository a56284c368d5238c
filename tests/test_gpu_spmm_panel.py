"""Sparse product of matrices with many entries a row (column panels, several entries per gather) against the oracle:
widths around the panel edges, every storage type and epilogue, rows of every length class, unaligned operands."""
import numpy as np
import pytest
import torch

import oracle
import paper_2604_02651_amd as sg
from gpu_util import DEV, TOL_F32, ctx, dev, rel_err

pytestmark = pytest.mark.gpu
ROWS, COLS = 1100, 20000
# fp32 sums of up to 17000 terms, rounded once to bfloat16 where the result is stored so
TOL_OUT = {torch.float32: TOL_F32, torch.bfloat16: 2.0 ** -8}


@pytest.fixture(scope="module")
def matrix():
    rng = np.random.default_rng(5)
    lens = rng.integers(0, 180, ROWS)
    lens[[0, 7, 8, 100, 1099]] = 0                                            # empty rows, the first and the last among them
    # one entry, a full fetch and one more, an item of a long row and one more, several items, longer pieces
    lens[[1, 2, 3, 20, 21, 22, 60, 61, 62]] = [1, 64, 65, 1024, 1025, 2048, 3000, 17000, 16385]
    ci = np.concatenate([np.sort(rng.choice(COLS, n, replace=False)).astype(np.int32) for n in lens])
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    assert len(ci) >= 40 * ROWS + 65536          # the launcher's rule
    return rp, ci, rng.standard_normal(len(ci)).astype(np.float32)


def _operand(rows, d, dtype, ld, seed, offset=0):
    """rows x d view with leading dimension ld that starts `offset` elements behind an aligned address."""
    gen = torch.Generator().manual_seed(seed)
    flat = torch.randn(rows * ld + offset, generator=gen).to(dtype).to(DEV)
    return flat[offset:].view(rows, ld)[:, :d]


def _np(t):
    return t.double().cpu().numpy()


@pytest.mark.parametrize("x_dtype,d", [(torch.float32, d) for d in (4, 31, 32, 33, 47, 64, 65, 128, 129, 256, 300, 602)] +
                         [(torch.bfloat16, d) for d in (8, 33, 64, 65, 128, 172, 256, 257, 510)])
def test_widths(matrix, x_dtype, d):
    rp, ci, v = matrix
    A = sg.Csr.from_arrays(ROWS, COLS, rp, ci, v, DEV, with_plan=d % 2 == 0)
    if A.plan is not None:
        sg.sgnn_csr_plan(ctx(), A)
    X = _operand(COLS, d, x_dtype, d + d % 3, d, offset=d % 5)
    ref = oracle.spmm(rp, ci, v, _np(X))
    out = torch.full((ROWS + 1, d), 7.0, device=DEV)
    sg.sgnn_spmm(ctx(), A, X, out[:ROWS])
    assert rel_err(out[:ROWS].cpu().numpy(), ref) < TOL_F32
    assert torch.all(out[ROWS] == 7.0)
    again = torch.empty_like(out)
    sg.sgnn_spmm(ctx(), A, X, again[:ROWS])                                  # the tickets are back where they were
    assert torch.equal(again[:ROWS], out[:ROWS])
    # through a row index (64-bit offsets), the result stored as bfloat16, a matrix added
    perm = np.random.default_rng(d).permutation(COLS).astype(np.int32)
    inv = torch.empty(COLS, dtype=torch.int64, device=DEV)
    inv[dev(perm).long()] = torch.arange(COLS, device=DEV)
    out16 = torch.empty((ROWS, d + (3 if d <= 512 else 2)), dtype=torch.bfloat16, device=DEV)[:, :d]
    add = _operand(ROWS, d, torch.float32, d + 4, 3)
    sg.sgnn_spmm(ctx(), A, X[inv].contiguous(), out16, row_index=dev(perm), add=add)
    assert rel_err(_np(out16), ref + _np(add)) < TOL_OUT[torch.bfloat16]


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("d", [40, 47, 200])
def test_layer_epilogues(matrix, d, bf16):
    # bias and ReLU of a transform-first layer, and the ReLU mask of the layer below in the transposed product
    rp, ci, v = matrix
    n, ci = ROWS, ci % ROWS                                                  # square: the columns folded together
    A = sg.Csr.from_arrays(n, n, rp, ci, v, DEV)
    ctx().reserve(n, len(ci), n, 256, len(ci))
    act = torch.bfloat16 if bf16 else torch.float32
    tol = 2e-2 if bf16 else TOL_F32
    flags = sg.SGNN_RELU | (sg.SGNN_BF16_MFMA if bf16 else 0)
    d_in = d + 24
    H, W, b = _operand(n, d_in, act, d_in, 1), _operand(d_in, d, torch.float32, d, 2), _operand(1, d, torch.float32, d, 3)[0]
    Y = torch.empty((n, d), dtype=act, device=DEV)
    sg.sgnn_gcn_fwd(ctx(), A, H, W, b, flags | sg.SGNN_XFORM_FIRST, Y, None)
    ref = np.maximum(oracle.spmm(rp, ci, v, _np(H) @ _np(W)) + _np(b), 0)
    assert rel_err(_np(Y), ref) < tol
    dY, Hin = _operand(n, d_in, act, d_in, 4), _operand(n, d, act, d, 5)
    T, dH, W2 = _operand(n, d, act, d, 6), torch.empty((n, d), dtype=act, device=DEV), _operand(d, d_in, torch.float32, d_in, 7)
    sg.sgnn_gcn_bwd(ctx(), A, T, W2, None, dY, flags | sg.SGNN_DY_MASKED, dH, None, None, H_in=Hin)
    ref = oracle.spmm(rp, ci, v, _np(dY) @ _np(W2).T) * (_np(Hin) > 0)
    assert rel_err(_np(dH), ref) < tol


@pytest.mark.parametrize("mean", [0, 3, 11, 12])
def test_room_for_more_entries_than_there_are(mean):
    # the host sees the capacity, the device the entries: both kernels are launched and the one for short rows does the work
    rows, cap = 900, 130000
    rng = np.random.default_rng(mean)
    lens = np.full(rows, mean)
    lens[[3, 50]] = [300, 2000] if mean else 0
    lens[60:60 + (2300 - 2 * mean if mean else 0) // 10] -= min(mean, 10)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ci = rng.integers(0, rows, rp[-1]).astype(np.int32)
    v = rng.standard_normal(len(ci)).astype(np.float32)
    A = sg.Csr(rows, rows, cap, DEV)
    A.rowptr.copy_(torch.as_tensor(rp))
    A.colidx[:len(ci)] = dev(ci)
    A.val[:len(ci)] = dev(v)
    sg.sgnn_csr_plan(ctx(), A)
    X = _operand(rows, 100, torch.float32, 100, mean)
    out = torch.full((rows, 100), 7.0, device=DEV)
    sg.sgnn_spmm(ctx(), A, X, out)
    assert rel_err(out.cpu().numpy(), oracle.spmm(rp, ci, v, _np(X))) < TOL_F32


@pytest.mark.parametrize("rows,d,mean", [(32768, 47, 12), (32768, 47, 13), (32768, 127, 13), (32767, 128, 13), (32768, 128, 13), (32768, 128, 31), (32768, 128, 32)])
def test_either_side_of_the_limit(rows, d, mean):
    # room for 40 entries a row and 65536 more: the device decides by the mean (for these widths the limits are those of the next test)
    rng = np.random.default_rng(mean)
    lens = np.full(rows, mean)
    lens[5], lens[10:10 + 900] = lens[5] + 900, lens[10:10 + 900] - 1
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ci = rng.integers(0, rows, rp[-1]).astype(np.int32)
    v = rng.standard_normal(len(ci)).astype(np.float32)
    A = sg.Csr(rows, rows, 40 * rows + 65536, DEV)
    A.rowptr.copy_(torch.as_tensor(rp))
    A.colidx[:len(ci)] = dev(ci)
    A.val[:len(ci)] = dev(v)
    sg.sgnn_csr_plan(ctx(), A)
    X = _operand(rows, d, torch.float32, d, mean)
    out = torch.full((rows, d), 7.0, device=DEV)
    sg.sgnn_spmm(ctx(), A, X, out)
    assert rel_err(out.cpu().numpy(), oracle.spmm(rp, ci, v, _np(X))) < TOL_F32


def _with_mean(rows, cols, mean, capacity, seed):
    """rows x cols with exactly rows * mean entries, rows of different lengths, and room for `capacity`."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    lens = torch.full((rows,), mean, device=DEV)
    lens[5] += 900
    lens[10:910] -= 1
    A = sg.Csr(rows, cols, capacity, DEV)
    A.rowptr[1:] = lens.cumsum(0)
    n = rows * mean
    A.colidx[:n] = torch.randint(0, cols, (n,), generator=gen, device=DEV, dtype=torch.int32)
    A.val[:n] = torch.randn(n, generator=gen, device=DEV)
    sg.sgnn_csr_plan(ctx(), A)
    return A


@pytest.mark.parametrize("rows,cols,x_dtype,d,add,limit", [
    (2499, 2499, torch.float32, 47, False, 56), (2500, 2500, torch.float32, 47, False, 16), (2500, 9000, torch.float32, 32, False, 10),
    (6499, 6499, torch.bfloat16, 64, False, 36), (6499, 6499, torch.bfloat16, 65, False, 64), (6500, 6500, torch.bfloat16, 64, False, 16),
    (8192, 8192, torch.float32, 64, False, 12), (8192, 8192, torch.bfloat16, 129, False, 46), (8192, 8192, torch.bfloat16, 257, False, 44),
    (16999, 16999, torch.bfloat16, 128, False, 12), (17000, 17000, torch.bfloat16, 128, False, 30), (22499, 5000, torch.float32, 65, False, 32),
    (40000, 40000, torch.float32, 100, False, 40), (44999, 44999, torch.float32, 256, False, 35),
    (45000, 45000, torch.float32, 129, False, 32), (61999, 61999, torch.float32, 65, False, 32), (62000, 62000, torch.float32, 128, False, 28),
    (65536, 65536, torch.bfloat16, 47, False, 38), (119999, 119999, torch.bfloat16, 256, False, 32), (120000, 120000, torch.bfloat16, 256, False, 24),
    (120000, 120000, torch.float32, 64, False, 30), (131072, 131072, torch.bfloat16, 400, False, 20), (262144, 262144, torch.float32, 256, False, 20),
    # three panels, or a matrix added that is not in whole 16 bytes: the other kernel is the main one
    (32767, 32767, torch.float32, 300, False, 13), (32768, 32768, torch.float32, 300, False, 32), (32768, 100000, torch.float32, 300, False, 13),
    (32768, 32768, torch.float32, 47, True, 13)])
def test_which_kernel_works(rows, cols, x_dtype, d, add, limit):
    # Both kernels are launched.  Below the limit the result is bit for bit the one of the other kernel alone (a matrix without room for 40
    # entries a row, 60 under 8192 rows, is not launched for the panel kernel); from the limit on the sums have another order.
    room = (60 if rows < 8192 else 40) * rows + 65536
    X = _operand(cols, d, x_dtype, d, 1)
    extra = _operand(rows, d, torch.float32, d + 1, 2) if add else None
    ctx().reserve(rows, room, rows, 512, room)
    for mean in (limit - 1, limit):
        out = [torch.full((rows, d), 7.0, device=DEV) for _ in range(2)]
        for o, capacity in zip(out, (room, rows * mean)):
            assert (capacity < room) == (o is out[1])
            sg.sgnn_spmm(ctx(), _with_mean(rows, cols, mean, capacity, 3), X, o, add=extra)
        assert torch.equal(out[0], out[1]) == (mean < limit)
        # fp32 sums of at most 942 terms of a standard normal distribution, rel_err's bar as everywhere
        assert (out[0] - out[1]).norm() < TOL_F32 * out[1].norm() and (out[0] - out[1]).abs().max() < TOL_F32 * out[1].abs().max()


@pytest.mark.parametrize("x_dtype", [torch.float32, torch.bfloat16])
def test_infinities_stay_in_their_rows(matrix, x_dtype):
    # lanes without an entry of their own must not add 0 * x of somebody else's
    rp, ci, v = matrix
    A = sg.Csr.from_arrays(ROWS, COLS, rp, ci, v, DEV)
    X = _operand(COLS, 47, x_dtype, 48, 9)
    X[0] = float("inf")
    X[int(ci[-1]), 3] = float("nan")
    X[int(ci[5]), 46] = -float("inf")
    out = torch.empty((ROWS, 47), device=DEV)
    sg.sgnn_spmm(ctx(), A, X, out)
    with np.errstate(invalid="ignore"):
        ref = oracle.spmm(rp, ci, v, _np(X))
    got = _np(out)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    fine = np.isfinite(ref)
    assert rel_err(got[fine], ref[fine]) < TOL_F32


def test_rows_of_more_than_4_gb():
    rows, cols, d, ld = 900, 3, 40, (1 << 30) + 8
    rng = np.random.default_rng(11)
    rp = np.arange(rows + 1) * 150
    ci = rng.integers(0, cols, rp[-1]).astype(np.int32)
    v = rng.standard_normal(len(ci)).astype(np.float32)
    A = sg.Csr.from_arrays(rows, cols, rp, ci, v, DEV)
    X = torch.empty(cols * ld, device=DEV).view(cols, ld)[:, :d]
    X.copy_(torch.randn((cols, d), generator=torch.Generator().manual_seed(12)))
    out = torch.empty((rows, d), device=DEV)
    sg.sgnn_spmm(ctx(), A, X, out)
    assert rel_err(out.cpu().numpy(), oracle.spmm(rp, ci, v, _np(X))) < TOL_F32
    del X
    torch.cuda.empty_cache()
