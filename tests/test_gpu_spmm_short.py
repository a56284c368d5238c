"""Sparse product of matrices with few entries a row (a stream of rows for every group of lanes) against the oracle: widths around
the group and panel edges, every storage type and epilogue, rows of every length class, unaligned operands, 32-bit and 64-bit offsets."""
import numpy as np
import pytest
import torch

import oracle
import paper_2604_02651_amd as sg
from gpu_util import DEV, TOL_F32, ctx, dev, fail_next_launch, rel_err
from test_gpu_spmm_panel import TOL_OUT, _np, _operand

pytestmark = pytest.mark.gpu


def _csr(lens, cols, seed):
    rng = np.random.default_rng(seed)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ci = rng.integers(0, cols, rp[-1]).astype(np.int32)
    return rp, ci, rng.standard_normal(len(ci)).astype(np.float32)


def _few_pieces():
    # pieces shared by the groups of a wavefront: empty rows (first, last, whole blocks), pieces of 1, 63 and 64 entries, two pieces,
    # more than 64 pieces (two to a partial row), more than 256 (longer pieces)
    lens = np.random.default_rng(1).integers(0, 9, 3001)
    lens[[0, 3000]] = 0
    lens[100:180] = 0
    lens[[1, 2, 50, 51, 52, 53, 54, 700, 1500]] = [65, 64, 63, 128, 129, 300, 9, 4097, 17000]
    return lens


def _many_pieces():
    # a piece for every group: more than 4096 of them
    lens = np.random.default_rng(2).integers(0, 3, 40001)
    lens[np.random.default_rng(3).permutation(40001)[:4500]] = 16
    lens[[5, 6, 39999]] = [200, 65, 5000]
    return lens


def _hubs():
    # few pieces, some of rows of 64 partial rows and more: pieces of 64, 128, 256 and 512 entries
    lens = np.random.default_rng(5).integers(0, 9, 20001)
    lens[[7, 8, 3000, 20000]] = [10000, 17000, 40000, 100000]
    return lens


def _pieces(lens):
    # pieces of long rows, those of more than four times the mean (and eight): 64 entries, doubled until a row has 256 of them at most
    long = lens[lens > max(4 * (lens.sum() // len(lens)), 8)]
    return sum(-(-n // next(c for c in (64 << i for i in range(20)) if n <= 256 * c)) for n in long)


def _hubs_and_many_pieces():
    lens = _many_pieces()
    lens[lens == 16] = 48
    lens[[7, 8, 3000, 40000]] = [10000, 17000, 40000, 100000]
    assert _pieces(lens) >= 4096             # a piece for every group of lanes
    return lens


def _blocks(lens, groups, panels=1):
    """Rows that are not long of every block of a wavefront of so many groups: what a block walks, and with the long ones in place."""
    mean, long_len = lens.sum() // len(lens), max(4 * (lens.sum() // len(lens)), 8)
    rows = min(max(min(48 // mean, len(lens) * panels // (4096 * groups)), 1), 8) * groups
    lens = np.pad(lens, (0, -len(lens) % rows)).reshape(-1, rows)
    return np.where(lens > long_len, 0, lens).sum(1), (lens > long_len).any(1), (lens == 0).any(1)


def _blocks_in_parts(low, high, row, *shapes):
    # rows of the length up to which they do not count as long side by side: the entries of a block do not fit the part of LDS they go
    # through, a row begins in one part and ends in the next, with empty rows and long ones in such blocks too
    lens = np.random.default_rng(4).integers(low, high, 40001)
    lens[1000:3000] = row
    lens[1003:3000:37] = 0
    lens[1018:3000:37] = 300
    for groups, panels, entries in shapes:
        walked, has_long, has_empty = _blocks(lens, groups, panels)
        parts = walked > entries
        assert (parts & has_long).any() and (parts & has_empty).any() and (parts & ~has_long & ~has_empty).any()
    return lens


def _full_blocks():
    return _blocks_in_parts(14, 19, 76, (8, 1, 512), (4, 1, 512))       # groups of 8 and of 16 lanes: 512 entries in LDS at a time


def _full_wide_blocks():
    return _blocks_in_parts(8, 13, 48, (2, 1, 256), (2, 2, 256))        # groups of 32 lanes: 256


MATRICES = {"few": _few_pieces, "many": _many_pieces, "full": _full_blocks, "full_wide": _full_wide_blocks}
HUBS = {"hubs": _hubs, "hubs_many": _hubs_and_many_pieces}


@pytest.mark.parametrize("name", MATRICES)
@pytest.mark.parametrize("x_dtype,d", [(torch.float32, d) for d in (4, 31, 32, 33, 64, 65, 128, 129, 200, 256)] +
                         [(torch.bfloat16, d) for d in (8, 47, 64, 65, 128, 129, 256, 257, 510)])
def test_widths(name, x_dtype, d):
    lens, cols = MATRICES[name](), 2500
    rows = len(lens)
    rp, ci, v = _csr(lens, cols, d)
    A = sg.Csr.from_arrays(rows, cols, rp, ci, v, DEV, with_plan=d % 2 == 0)
    if A.plan is not None:
        sg.sgnn_csr_plan(ctx(), A)
    ctx().reserve(rows, len(ci), rows, 512, len(ci))
    X = _operand(cols, d, x_dtype, d + d % 3, d, offset=d % 5)
    ref = oracle.spmm(rp, ci, v, _np(X))
    out = torch.full((rows + 1, d), 7.0, device=DEV)
    sg.sgnn_spmm(ctx(), A, X, out[:rows])
    assert rel_err(out[:rows].cpu().numpy(), ref) < TOL_F32
    assert torch.all(out[rows] == 7.0)
    again = torch.empty_like(out)
    sg.sgnn_spmm(ctx(), A, X, again[:rows])                                  # the tickets are back where they were
    assert torch.equal(again[:rows], out[:rows])
    # through a row index (64-bit offsets), the result stored as bfloat16; a matrix added, in whole 16 bytes and not
    perm = np.random.default_rng(d).permutation(cols).astype(np.int32)
    inv = torch.empty(cols, dtype=torch.int64, device=DEV)
    inv[dev(perm).long()] = torch.arange(cols, device=DEV)
    out16 = torch.empty((rows, d + 3), dtype=torch.bfloat16, device=DEV)[:, :d]
    sg.sgnn_spmm(ctx(), A, X[inv].contiguous(), out16, row_index=dev(perm))
    assert rel_err(_np(out16), ref) < TOL_OUT[torch.bfloat16]
    for ld in (d + 4, d + 5):
        add = _operand(rows, d, torch.float32, ld, 3)
        sg.sgnn_spmm(ctx(), A, X, out[:rows], add=add)
        assert rel_err(out[:rows].cpu().numpy(), ref + _np(add)) < TOL_F32


@pytest.mark.parametrize("name", HUBS)
@pytest.mark.parametrize("x_dtype,d", [(torch.float32, 33), (torch.float32, 200), (torch.bfloat16, 47), (torch.bfloat16, 256), (torch.bfloat16, 400)])
def test_hub_rows(name, x_dtype, d):
    lens, cols = HUBS[name](), 2500
    rows = len(lens)
    rp, ci, v = _csr(lens, cols, d)
    A = sg.Csr.from_arrays(rows, cols, rp, ci, v, DEV, with_plan=True)
    ctx().reserve(rows, len(ci), rows, 512, len(ci))
    X = _operand(cols, d, x_dtype, d, d)
    ref = oracle.spmm(rp, ci, v, _np(X))
    first = None
    for _ in range(3):
        sg.sgnn_csr_plan(ctx(), A)                                           # the pieces are numbered anew
        out = torch.full((rows, d), 7.0, device=DEV)
        sg.sgnn_spmm(ctx(), A, X, out)
        assert rel_err(out.cpu().numpy(), ref) < TOL_F32
        first = out if first is None else first
        assert torch.equal(out, first)


def _few_rows(rows):
    # few rows of many entries, of very different lengths: the groups of a wavefront share every row.  Empty rows (first, last, side by side), one
    # entry, a full fetch and one more, rows just under and over the length from which they count as long (four times the mean), a hub
    lens = np.random.default_rng(rows).integers(0, 120, rows)
    lens[[0, rows - 1]] = 0
    lens[10:20] = 0
    lens[[1, 2, 3, 4, 5, 6, 7, 8]] = [1, 8, 9, 63, 64, 65, 128, 129]
    lens[[30, 31, 32, 33]] = [236, 237, 300, 5000]
    return lens


@pytest.mark.parametrize("rows", [257, 1024, 1500])
@pytest.mark.parametrize("x_dtype,d", [(torch.float32, 4), (torch.float32, 47), (torch.float32, 128), (torch.float32, 200),
                                       (torch.bfloat16, 8), (torch.bfloat16, 47), (torch.bfloat16, 100), (torch.bfloat16, 256), (torch.bfloat16, 257)])
def test_few_rows_of_many_entries(rows, x_dtype, d):
    lens, cols = _few_rows(rows), 2500
    assert rows < 7 * (lens.sum() // rows) * 8                                # 8: the fewest values a wavefront adds up side by side
    rp, ci, v = _csr(lens, cols, d)
    A = sg.Csr.from_arrays(rows, cols, rp, ci, v, DEV, with_plan=True)
    assert A.capacity < 60 * rows + 65536                                     # not launched for the panel kernel as well
    ctx().reserve(rows, len(ci), rows, 512, len(ci))
    X = _operand(cols, d, x_dtype, d + d % 3, d, offset=d % 5)
    ref = oracle.spmm(rp, ci, v, _np(X))
    first = None
    for _ in range(2):
        sg.sgnn_csr_plan(ctx(), A)
        out = torch.full((rows + 1, d), 7.0, device=DEV)
        sg.sgnn_spmm(ctx(), A, X, out[:rows])
        assert rel_err(out[:rows].cpu().numpy(), ref) < TOL_F32
        assert torch.all(out[rows] == 7.0)
        first = out if first is None else first
        assert torch.equal(out, first)
    perm = np.random.default_rng(d).permutation(cols).astype(np.int32)
    inv = torch.empty(cols, dtype=torch.int64, device=DEV)
    inv[dev(perm).long()] = torch.arange(cols, device=DEV)
    sg.sgnn_spmm(ctx(), A, X[inv].contiguous(), out[:rows], row_index=dev(perm))
    assert rel_err(out[:rows].cpu().numpy(), ref) < TOL_F32
    add = _operand(rows, d, torch.float32, d + 4, 3)
    sg.sgnn_spmm(ctx(), A, X, out[:rows], add=add)
    assert rel_err(out[:rows].cpu().numpy(), ref + _np(add)) < TOL_F32


@pytest.mark.parametrize("x_dtype,d", [(torch.float32, 40), (torch.bfloat16, 48), (torch.bfloat16, 100)])
def test_few_rows_are_added_up_in_short_chains(x_dtype, d):
    # rows of 400 entries, see the next test: every group of lanes has its share of each fetch of 64, a half of it where rows of X are widest
    rows, n = 1000, 400
    ci = np.random.default_rng(1).integers(1, rows, rows * n).astype(np.int32)
    ci[::n] = 0
    A = sg.Csr.from_arrays(rows, rows, np.arange(rows + 1) * n, ci, np.ones(rows * n, np.float32), DEV, with_plan=True)
    X = torch.ones((rows, d), device=DEV, dtype=x_dtype)
    X[0] = 2.0 ** 24
    out = torch.empty((rows, d), device=DEV)
    y, loss = torch.zeros(rows, dtype=torch.int32, device=DEV), torch.zeros(1, device=DEV)
    sg.sgnn_csr_plan(ctx(), A)
    sg.sgnn_spmm_xent(ctx(), A, X, None, y, loss, None, O=out)
    missing = 2.0 ** 24 + n - 1 - out.double()
    assert torch.all(missing >= -2) and torch.all(missing <= n // 2 + 32)


@pytest.mark.parametrize("x_dtype,d", [(torch.float32, 40), (torch.float32, 100), (torch.bfloat16, 48), (torch.bfloat16, 256)])
def test_long_rows_are_added_up_in_short_chains(x_dtype, d):
    # a row of 1e5 entries in a matrix with a piece for every group of lanes: pieces of 512 entries, a chain of gathers each.  A chain
    # that begins with 2^24 loses every one after it (2^24 + 1 rounds to 2^24), the others are exact: what is missing is the chain's length.
    lens, cols = _hubs_and_many_pieces(), 2500
    lens[[7, 8, 3000, 40000, 77]] = [1, 1, 1, 1, 100000]
    assert _pieces(lens) >= 4096
    rows = len(lens)
    rp, ci, v = _csr(lens, cols, 1)
    ci[ci == 0] = 1
    ci[rp[77]] = 0
    v[:] = 1
    A = sg.Csr.from_arrays(rows, cols, rp, ci, v, DEV)
    X = torch.ones((cols, d), device=DEV, dtype=x_dtype)
    X[0] = 2.0 ** 24
    out = torch.empty((rows, d), device=DEV)
    sg.sgnn_spmm(ctx(), A, X, out)
    missing = 2.0 ** 24 + 99999 - out[77].double()
    assert torch.all(missing >= -2) and torch.all(missing <= 512 + 2)        # 2: sums over 2^24 are even
    out[77] = 0
    assert torch.equal(out.cpu(), torch.as_tensor(np.where(np.arange(rows) == 77, 0, lens), dtype=torch.float32)[:, None].expand(rows, d))


@pytest.mark.parametrize("name", [*MATRICES, "few_rows"])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("d", [40, 47, 200])
def test_layer_epilogues(name, d, bf16):
    # bias and ReLU of a transform-first layer, and the ReLU mask of the layer below in the transposed product
    lens = MATRICES[name]() if name in MATRICES else _few_rows(1024)
    n = len(lens)
    rp, ci, v = _csr(lens, n, d)
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


@pytest.mark.parametrize("x_dtype", [torch.float32, torch.bfloat16])
def test_infinities_stay_in_their_rows(x_dtype):
    lens, cols = _few_pieces(), 2500
    rp, ci, v = _csr(lens, cols, 9)
    A = sg.Csr.from_arrays(len(lens), cols, rp, ci, v, DEV)
    X = _operand(cols, 47, x_dtype, 48, 9)
    X[0] = float("inf")
    X[int(ci[-1]), 3] = float("nan")
    X[int(ci[5]), 46] = -float("inf")
    out = torch.empty((len(lens), 47), device=DEV)
    sg.sgnn_spmm(ctx(), A, X, out)
    with np.errstate(invalid="ignore"):
        ref = oracle.spmm(rp, ci, v, _np(X))
    got = _np(out)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    fine = np.isfinite(ref)
    assert rel_err(got[fine], ref[fine]) < TOL_F32


@pytest.mark.parametrize("name", [*MATRICES, *HUBS, "few_rows"])
@pytest.mark.parametrize("x_dtype,d", [(torch.float32, d) for d in (4, 7, 32, 33, 64, 66, 100, 128)] +
                         [(torch.bfloat16, d) for d in (8, 47, 64, 66, 128, 132, 172, 256)])
def test_loss_in_the_epilogue(name, x_dtype, d):
    lens = {**MATRICES, **HUBS, "few_rows": lambda: _few_rows(1024)}[name]()
    n = len(lens)
    rp, ci, v = _csr(lens, n, d)
    v = v * np.float32(0.1)      # logits of a few units: exp(x - max) keeps the tolerance of the product
    A = sg.Csr.from_arrays(n, n, rp, ci, v, DEV, with_plan=True)
    ctx().reserve(n, len(ci), n, 256, len(ci))
    X, b = _operand(n, d, x_dtype, d + 4 - d % 4, d), _operand(1, d, torch.float32, d, 3)[0]
    y = np.random.default_rng(d).integers(0, d, n).astype(np.int32)
    y[[0, 40, n - 1]] = [d - 1, 0, d]                                         # the last: no class, the log-sum-exp alone
    O = oracle.spmm(rp, ci, v, _np(X)) + _np(b)
    m = O.max(1, keepdims=True)
    e = np.exp(O - m)
    s = e.sum(1, keepdims=True)
    inside = y < d
    hit = np.zeros_like(O)
    hit[np.arange(n)[inside], y[inside]] = 1
    dO_ref = (e / s - hit) / n
    loss_ref = ((m + np.log(s))[:, 0] - (O * hit).sum(1)).mean()
    bf16 = x_dtype == torch.bfloat16
    first = None
    for keep in (True, False, False):
        sg.sgnn_csr_plan(ctx(), A)                                            # the pieces are numbered anew
        loss, db = torch.zeros(1, device=DEV), torch.empty(d, device=DEV)
        dO = torch.full((n + 1, d + 4 - d % 4), 7.0, dtype=x_dtype, device=DEV)[:, :d]
        logits = torch.empty((n, d), device=DEV) if keep else None
        sg.sgnn_spmm_xent(ctx(), A, X, b, dev(y), loss, dO[:n], O=logits, dO_colsum=db)
        if keep:
            assert rel_err(_np(logits), O) < TOL_F32
        assert torch.all(dO[n] == 7.0)
        # one rounding of every entry where dO is bfloat16; the column sums add what is stored
        assert rel_err(_np(dO[:n]), dO_ref) < (2.0 ** -8 if bf16 else TOL_F32)
        got = _np(dO[:n])
        assert np.abs(_np(db) - got.sum(0)).max() < 1e-5 * np.abs(got).sum(0).max()
        assert abs(loss.item() - loss_ref) < TOL_F32 * abs(loss_ref)
        if first is None:
            first = (loss.clone(), db.clone(), dO.clone())
        assert torch.equal(loss, first[0]) and torch.equal(db, first[1]) and torch.equal(dO, first[2])


# six values a lane: from one column above half of a group's lanes' sixteen bytes to the last that six values cover, and one more
@pytest.mark.parametrize("name", ["few", "many", "full", "hubs", "few_rows"])
@pytest.mark.parametrize("d", [33, 46, 48, 49, 65, 95, 96, 97, 129, 131, 191, 192, 193])
def test_loss_with_six_values_a_lane(name, d):
    test_loss_in_the_epilogue(name, torch.bfloat16, d)


# widths and strides of no multiple, and a class that a bias takes out of the sums: its share is 0, the rest as without it
@pytest.mark.parametrize("x_dtype,d,ld", [(torch.float32, 67, 69), (torch.float32, 127, 127), (torch.bfloat16, 95, 97), (torch.bfloat16, 130, 131),
                                          (torch.bfloat16, 255, 255), (torch.bfloat16, 47, 47)])
@pytest.mark.parametrize("out", [-np.inf, -3.4e38])
def test_loss_at_any_stride_and_without_a_class(x_dtype, d, ld, out):
    lens = _few_pieces()
    n = len(lens)
    rp, ci, v = _csr(lens, n, d)
    v = v * np.float32(0.1)
    A = sg.Csr.from_arrays(n, n, rp, ci, v, DEV, with_plan=True)
    ctx().reserve(n, len(ci), n, 256, len(ci))
    sg.sgnn_csr_plan(ctx(), A)
    X = _operand(n, d, x_dtype, ld, d)
    b = torch.zeros(d, device=DEV)
    b[d // 2] = out
    y = np.random.default_rng(d).integers(0, d, n).astype(np.int32)
    y[y == d // 2] = 0
    O = oracle.spmm(rp, ci, v, _np(X))
    O[:, d // 2] = -np.inf
    m = O.max(1, keepdims=True)
    e = np.exp(O - m)
    s = e.sum(1, keepdims=True)
    dO_ref = e / s
    dO_ref[np.arange(n), y] -= 1
    dO_ref /= n
    loss_ref = ((m + np.log(s))[:, 0] - O[np.arange(n), y]).mean()
    loss, db = torch.zeros(1, device=DEV), torch.empty(d, device=DEV)
    dO = torch.full((n + 1, ld), 7.0, dtype=x_dtype, device=DEV)
    sg.sgnn_spmm_xent(ctx(), A, X, b, dev(y), loss, dO[:n, :d], dO_colsum=db)
    assert torch.all(dO[n] == 7.0) and torch.all(dO[:, d:] == 7.0) and torch.all(dO[:n, d // 2] == 0)
    got = _np(dO[:n, :d])
    assert rel_err(got, dO_ref) < (2.0 ** -8 if x_dtype == torch.bfloat16 else TOL_F32)
    assert np.abs(_np(db) - got.sum(0)).max() < 1e-5 * np.abs(got).sum(0).max()
    assert abs(loss.item() - loss_ref) < TOL_F32 * abs(loss_ref)


# Long rows add to the sums as integers: what is no finite number comes through all the same (both kernels, every piece length)
@pytest.mark.parametrize("name,row", [("few", 1500), ("many", 5), ("hubs", 20000)])
@pytest.mark.parametrize("x_dtype,d,ld", [(torch.float32, 47, 48), (torch.float32, 67, 69), (torch.float32, 300, 300), (torch.bfloat16, 47, 48),
                                          (torch.bfloat16, 95, 97), (torch.bfloat16, 172, 176)])
def test_long_row_that_is_not_finite(name, row, x_dtype, d, ld):
    lens = {**MATRICES, **HUBS}[name]()
    n = len(lens)
    rp, ci, v = _csr(lens, n, d)
    ctx().reserve(n, len(ci), n, 512, len(ci))
    X = _operand(n, d, x_dtype, ld, d)
    y = np.random.default_rng(d).integers(0, d - 1, n).astype(np.int32)

    def call(v, y, b):
        A = sg.Csr.from_arrays(n, n, rp, ci, v, DEV, with_plan=True)
        sg.sgnn_csr_plan(ctx(), A)
        loss, db, dO = torch.zeros(1, device=DEV), torch.zeros(d, device=DEV), torch.zeros((n, ld), dtype=x_dtype, device=DEV)[:, :d]
        sg.sgnn_spmm_xent(ctx(), A, X, b, dev(y), loss, dO, dO_colsum=db)
        return loss.item(), db, dO

    others = torch.arange(n, device=DEV) != row
    for bad in (np.nan, np.inf):
        w = v * np.float32(0.1)
        w[rp[row] + 1] = bad
        loss, db, dO = call(w, y, None)
        assert np.isnan(loss) and torch.isnan(db).all()
        assert torch.isnan(dO[row]).all() and torch.isfinite(dO[others]).all()
    # the row's label is a class of logit minus infinity: an infinite loss, a gradient of -1 / n there
    b, t = torch.zeros(d, device=DEV), y.copy()
    b[d - 1], t[row] = -np.inf, d - 1
    loss, db, dO = call(v * np.float32(0.1), t, b)
    assert loss == np.inf and torch.isfinite(db).all() and torch.isfinite(dO).all()
    assert abs(db[d - 1].item() * n + 1) < 2.0 ** -8


# The integer sums of long rows (both kernels) begin at zero whatever the call before wanted, at another width, and on every replay of a graph
@pytest.mark.parametrize("d", [47, 172, 300])
def test_loss_after_other_calls(d):
    lens = _hubs()
    n = len(lens)
    rp, ci, v = _csr(lens, n, 5)
    A = sg.Csr.from_arrays(n, n, rp, ci, v * np.float32(0.1), DEV, with_plan=True)
    ctx().reserve(n, len(ci), n, 512, len(ci))
    sg.sgnn_csr_plan(ctx(), A)
    y = dev(np.random.default_rng(d).integers(0, d, n).astype(np.int32))
    x = {w: _operand(n, w, torch.float32, w + 4 - w % 4, w) for w in (d, 64)}

    def call(c, w, loss, dO, db):
        out = [torch.full((1,), 3.0, device=DEV), torch.empty((n, w + 4 - w % 4), device=DEV)[:, :w], torch.full((w,), 3.0, device=DEV)]
        sg.sgnn_spmm_xent(c, A, x[w], None, y.clamp(max=w - 1), out[0] if loss else None, out[1] if dO else None, dO_colsum=out[2] if db else None)
        return out

    def context():
        c = sg.Context(0)
        c.reserve(n, len(ci), n, 512, len(ci))
        return c

    c = context()
    want = call(c, d, True, True, True)
    torch.cuda.synchronize()
    for other in ((d, True, False, False), (d, False, True, True), (64, False, True, False), (64, False, False, False), (d, True, True, True)):
        call(c, *other)
        got = call(c, d, True, True, True)
        assert [torch.equal(g, t) for g, t in zip(got, want)] == [True] * 3, other
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        got = call(c, d, True, True, True)
    for _ in range(3):
        for t in got:
            t.fill_(3.0)
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(g, t) for g, t in zip(got, want))
        again = call(c, d, True, True, True)
        torch.cuda.synchronize()
        assert all(torch.equal(g, t) for g, t in zip(again, want))
    c.close()


# A call that fails behind its product leaves nothing for later ones: a graph captured before it, one captured after it and not replayed yet, a call
@pytest.mark.parametrize("x_dtype,d", [(torch.float32, 47), (torch.bfloat16, 172), (torch.float32, 300)])
def test_loss_after_a_call_that_failed(x_dtype, d):
    lens = _hubs()
    n = len(lens)
    rp, ci, v = _csr(lens, n, 5)
    A = sg.Csr.from_arrays(n, n, rp, ci, v * np.float32(0.1), DEV, with_plan=True)
    c = sg.Context(0)
    c.reserve(n, len(ci), n, 512, len(ci))
    sg.sgnn_csr_plan(c, A)
    y = dev(np.random.default_rng(d).integers(0, d, n).astype(np.int32))
    X = _operand(n, d, x_dtype, d + 8 - d % 8, d)

    def call(out=None):
        out = out or [torch.full((1,), 3.0, device=DEV), torch.empty((n, d + 8 - d % 8), dtype=x_dtype, device=DEV)[:, :d], torch.full((d,), 3.0, device=DEV)]
        sg.sgnn_spmm_xent(c, A, X, None, y, out[0], out[1], dO_colsum=out[2])
        return out

    def captured():
        stream = torch.cuda.Stream()
        stream.wait_stream(torch.cuda.current_stream())
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            out = call()
        return graph, out

    want = call()

    def check(out):
        torch.cuda.synchronize()
        assert all(torch.equal(g, t) for g, t in zip(out, want))

    before, out_before = captured()
    spare = call()
    fail_next_launch(lambda: call(spare))
    before.replay()
    check(out_before)
    fail_next_launch(lambda: call(spare))
    after, out_after = captured()
    check(call())
    for _ in range(3):
        after.replay()
        check(out_after)
        check(call())
    c.close()


def _products(call, entries):
    """The sparse-product kernels of a call in a context with scratch for so many entries; None where it refuses for want of scratch."""
    c = sg.Context(0)
    try:
        c.reserve(1, 1, 1, 1, entries)
        c.profile(True)
        try:
            call(c)
        except sg.SgnnError as e:
            assert "scratch too small" in str(e)
            return None
        return [name for name, *_ in c.profile_read() if name in ("spmm_main_kernel", "spmm_short_kernel")]
    finally:
        c.close()


def _least_scratch(wanted):
    """The smallest number of entries that a bisection finds to satisfy `wanted`."""
    low, high = 0, 1 << 22
    assert not wanted(low) and wanted(high)
    while high - low > 1:
        mid = (low + high) // 2
        low, high = (low, mid) if wanted(mid) else (mid, high)
    return high


@pytest.mark.parametrize("with_plan", [False, True])
def test_scratch_for_the_main_kernel_only(with_plan):
    # partial rows of 129 columns: three times 64 in the main kernel where rows are not aligned, two panels of 128 here
    lens, cols, d = _few_pieces(), 2500, 129
    rows = len(lens)
    rp, ci, v = _csr(lens, cols, 1)
    A = sg.Csr.from_arrays(rows, cols, rp, ci, v, DEV, with_plan=with_plan)
    if with_plan:
        sg.sgnn_csr_plan(ctx(), A)
    X = _operand(cols, d, torch.float32, d, 1)
    ref = oracle.spmm(rp, ci, v, _np(X))
    out = torch.empty((rows, d), device=DEV)
    call = lambda c: sg.sgnn_spmm(c, A, X, out)
    least = _least_scratch(lambda n: _products(call, n) is not None)
    for entries, kernel in ((least, "spmm_main_kernel"), (_least_scratch(lambda n: _products(call, n) == ["spmm_short_kernel"]), "spmm_short_kernel")):
        out.fill_(7)
        assert _products(call, entries) == [kernel]
        assert rel_err(_np(out), ref) < TOL_F32


@pytest.mark.parametrize("x_dtype,d", [(torch.float32, 47), (torch.float32, 100), (torch.bfloat16, 47), (torch.bfloat16, 100), (torch.bfloat16, 172)])
@pytest.mark.parametrize("entries", [8, 100001])
def test_loss_of_the_main_kernel(x_dtype, d, entries):
    # a matrix of eight entries at most has no long rows and no plan; with 1e5 rows of one entry the main kernel leaves fewer partial sums than
    # the other and takes the call where there is scratch for those only
    n = min(entries * 500, 100001)
    rp = np.minimum(np.arange(n + 1) * entries // n, entries)
    rng = np.random.default_rng(d)
    ci, v = rng.integers(0, n, entries).astype(np.int32), rng.standard_normal(entries).astype(np.float32)
    A = sg.Csr.from_arrays(n, n, rp, ci, v, DEV, with_plan=True)
    sg.sgnn_csr_plan(ctx(), A)
    X, b = _operand(n, d, x_dtype, d + 4 - d % 4, d), _operand(1, d, torch.float32, d, 3)[0]
    y = rng.integers(0, d, n)
    O = torch.as_tensor(oracle.spmm(rp, ci, v, _np(X)) + _np(b))
    dO_ref = (torch.softmax(O, 1) - torch.nn.functional.one_hot(torch.as_tensor(y), d)) / n
    loss_ref = torch.nn.functional.cross_entropy(O, torch.as_tensor(y)).item()
    loss, db, dO = torch.zeros(1, device=DEV), torch.empty(d, device=DEV), torch.empty((n, d + 4 - d % 4), dtype=x_dtype, device=DEV)[:, :d]
    call = lambda c: sg.sgnn_spmm_xent(c, A, X, b, dev(y.astype(np.int32)), loss, dO, dO_colsum=db)
    scratch = 1 << 22 if entries == 8 else _least_scratch(lambda k: _products(call, k) is not None)
    loss.zero_()
    dO.fill_(7)
    assert _products(call, scratch) == ["spmm_main_kernel"]
    assert entries == 8 or _products(call, 1 << 22) == ["spmm_short_kernel"]
    got = _np(dO)
    # one rounding of every entry where dO is bfloat16; the column sums add what is stored
    assert rel_err(got, dO_ref.numpy()) < (2.0 ** -8 if x_dtype == torch.bfloat16 else TOL_F32)
    assert np.abs(_np(db) - got.sum(0)).max() < 1e-5 * np.abs(got).sum(0).max()
    assert abs(loss.item() - loss_ref) < TOL_F32 * abs(loss_ref)


@pytest.mark.parametrize("x_dtype,d", [(torch.float32, 47), (torch.float32, 128), (torch.bfloat16, 47), (torch.bfloat16, 100), (torch.bfloat16, 172)])
def test_loss_with_rows_of_x_beyond_4_gb(x_dtype, d):
    lens, cols = _few_pieces(), (1 << 20) + 77
    n, ld = len(lens), 4096
    rp, ci, v = _csr(lens, cols, d)
    v = v * np.float32(0.1)
    assert int(ci.max()) * ld * x_dtype.itemsize > 1 << 32
    A = sg.Csr.from_arrays(n, cols, rp, ci, v, DEV, with_plan=True)
    sg.sgnn_csr_plan(ctx(), A)
    ctx().reserve(n, len(ci), n, 256, len(ci))
    X = torch.empty((cols, ld), dtype=x_dtype, device=DEV)[:, :d]
    X.copy_(torch.randn((cols, d), generator=torch.Generator(device=DEV).manual_seed(d), device=DEV))
    y = np.random.default_rng(d).integers(0, d, n)
    O = torch.as_tensor(oracle.spmm(rp, ci, v, _np(X)))
    dO_ref = (torch.softmax(O, 1) - torch.nn.functional.one_hot(torch.as_tensor(y), d)) / n
    loss_ref = torch.nn.functional.cross_entropy(O, torch.as_tensor(y)).item()
    loss, db, dO = torch.zeros(1, device=DEV), torch.empty(d, device=DEV), torch.empty((n, d + 4 - d % 4), dtype=x_dtype, device=DEV)[:, :d]
    sg.sgnn_spmm_xent(ctx(), A, X, None, dev(y.astype(np.int32)), loss, dO, dO_colsum=db)
    got = _np(dO)
    assert rel_err(got, dO_ref.numpy()) < (2.0 ** -8 if x_dtype == torch.bfloat16 else TOL_F32)
    assert np.abs(_np(db) - got.sum(0)).max() < 1e-5 * np.abs(got).sum(0).max()
    assert abs(loss.item() - loss_ref) < TOL_F32 * abs(loss_ref)
