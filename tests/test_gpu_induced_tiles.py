"""Tiles of the induced-matrix passes: rows that start and end on tile edges, row tables at and over their size,
runs of empty rows, hub rows over several tiles - against the CPU oracle, bit-exact on indices."""
import numpy as np
import pytest
import torch

import oracle
import paper_2604_02651_amd as sg
from gpu_util import DEV, TOL_VAL, bitmap_rank_from_sample, ctx, gpu_sample

pytestmark = pytest.mark.gpu


def _lengths(kind):
    # a tile is 2048 entries, its row table holds 1025 rows
    r = np.random.default_rng(7)
    if kind == "ones":                                   # 2048 rows a tile: more than the table holds
        return np.full(9000, 1)
    if kind == "twos":                                   # 1024 rows a tile and the first of the next: the table is full
        return np.full(6001, 2)
    if kind == "twos_shifted":                           # every tile starts inside a row
        return np.r_[1, np.full(6000, 2)]
    if kind == "over_by_one":                            # one row more than the table holds, then one fewer
        return np.r_[np.full(1023, 2), 1, 1, np.full(1022, 2), 3, 1, np.full(3000, 4)]
    if kind == "gaps":                                   # runs of empty rows longer than the table between rows with entries
        d = np.zeros(9000, np.int64)
        d[[0, 1, 1500, 1501, 4000, 8000]] = [700, 1348, 5, 2043, 2048, 1]
        return d
    if kind == "leading":                                # nothing before the last rows
        return np.r_[np.zeros(2000, np.int64), 3, 0, 0, 2045, 0, 2049, 0]
    if kind == "edges":                                  # starts and ends around tile edges, a hub over three tiles
        return np.r_[2047, 1, 2048, 2049, 2047, 6000, 1, np.zeros(5, np.int64), 63, 64, 65, np.zeros(70, np.int64), r.integers(0, 9, 3000)]
    return np.r_[r.integers(0, 4, 5000), r.integers(0, 200, 300)]      # mixed


@pytest.mark.parametrize("rp32", [False, True])
@pytest.mark.parametrize("kind", ["ones", "twos", "twos_shifted", "over_by_one", "gaps", "leading", "edges", "mixed"])
def test_tiles_against_oracle(kind, rp32):
    deg = _lengths(kind).astype(np.int64)
    N = max(len(deg), 7000)                              # rows of 6000 entries want as many columns
    deg = np.r_[deg, np.zeros(N - len(deg), np.int64)]
    rng = np.random.default_rng(3)
    full = np.flatnonzero(deg)                           # a column's weight wants its degree: none without entries
    cols = full if len(full) >= deg.max() else np.arange(N)
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    colidx = np.concatenate([np.sort(rng.choice(cols, d, replace=False)) for d in deg[full]]).astype(np.int32)
    E = len(colidx)
    val = None if len(full) >= deg.max() else rng.random(E).astype(np.float32) + 0.5
    rpd = torch.as_tensor(rowptr, dtype=torch.int32 if rp32 else torch.int64).to(DEV)
    cid = torch.as_tensor(colidx).to(DEV)
    vd = None if val is None else torch.as_tensor(val).to(DEV)
    ctx().reserve(N, E, N, 8, E)
    for B in (N, N - 1, N // 3):
        S, bm, rk = gpu_sample(N, B, 2, B)
        S_ref = oracle.sample_uniform(N, B, 2, B)
        for rg in ((0, N, 0, N), (N // 3, N - 5, 11, N // 2), (1, 2, 0, N)):
            out = sg.Csr(B, B, E, DEV)
            out.rowptr.fill_(-7)
            nnz = sg.sgnn_induced_csr_range(ctx(), N, rpd, cid, vd, S, B, bm, rk, *rg, out, want_nnz=True)
            rp, ci, v = oracle.induced_csr_range(N, rowptr, colidx, S_ref, *rg, val=val)
            assert nnz == len(ci) and np.array_equal(out.rowptr.cpu().numpy(), rp), (kind, B, rg)
            assert np.array_equal(out.colidx.cpu().numpy()[:nnz], ci), (kind, B, rg)
            got = out.val.cpu().numpy()[:nnz].astype(np.float64)
            assert np.all(np.abs(got - v) <= TOL_VAL * np.abs(v)), (kind, B, rg)
    ctx().status()


def _induced(N, rowptr, colidx, S, out, want=True):
    words, ranks = bitmap_rank_from_sample(N, S)
    to = lambda a, t: torch.as_tensor(np.asarray(a).astype(t)).to(DEV)
    return sg.sgnn_induced_csr(ctx(), N, to(rowptr, np.int64), to(colidx, np.int32), None, to(S, np.int32), len(S),
                               torch.as_tensor(words.view(np.int64)).to(DEV), to(ranks, np.int32), out, want_nnz=want)


def test_many_expected_tiles():
    # 1220 tiles are expected: the survivors of earlier tiles come from the prefix sum
    N, d = 5000, 500
    rng = np.random.default_rng(5)
    rowptr = np.arange(N + 1) * d
    colidx = np.sort(np.argpartition(rng.random((N, N), np.float32), d, axis=1)[:, :d], axis=1).ravel()
    ctx().reserve(N, N * d, N, 8, N * d)
    for B in (N, N - 3, 2000):
        S = np.sort(rng.choice(N, B, replace=False))
        out = sg.Csr(B, B, N * d, DEV)
        nnz = _induced(N, rowptr, colidx, S, out)
        rp, ci, v = oracle.induced_csr(N, rowptr, colidx, S)
        assert nnz == len(ci) and np.array_equal(out.rowptr.cpu().numpy(), rp) and np.array_equal(out.colidx.cpu().numpy()[:nnz], ci)
        assert np.all(np.abs(out.val.cpu().numpy()[:nnz] - v) <= TOL_VAL * np.abs(v))


def test_far_more_tiles_than_expected():
    # eight rows hold nearly all entries and all eight are sampled: 17 tiles expected, 8600 there, more than workgroups
    N, big, d = 4000, np.array([0, 7, 8, 1000, 1001, 2500, 3998, 3999]), 2200007
    rng = np.random.default_rng(6)
    deg = np.ones(N, np.int64)
    deg[big] = d
    rowptr = np.concatenate([[0], np.cumsum(deg)])
    colidx = rng.integers(0, N, rowptr[-1]).astype(np.int32)
    keep = np.isin(colidx, big)
    row = np.repeat(np.arange(N), deg)
    sel = keep & np.isin(row, big)
    rp = np.concatenate([[0], np.cumsum(np.bincount(np.searchsorted(big, row[sel]), minlength=8))])
    ci = np.searchsorted(big, colidx[sel])
    ctx().reserve(N, len(colidx), 8, 8, len(ci))
    out = sg.Csr(8, 8, len(ci), DEV)
    assert _induced(N, rowptr, colidx, big, out) == len(ci)
    assert np.array_equal(out.rowptr.cpu().numpy(), rp) and np.array_equal(out.colidx.cpu().numpy(), ci)
    ctx().status()


def test_groups_of_tiles_in_one_call_after_another():
    # more tiles than are added up one by one, two samples in turn: the counts of the groups start at zero in every call
    N, big, d = 4000, np.array([0, 7, 8, 1000, 1001, 2500, 3998, 3999]), 2800003
    deg = np.ones(N, np.int64)
    deg[big] = d
    rowptr = np.concatenate([[0], np.cumsum(deg)])
    colidx = np.random.default_rng(7).integers(0, N, rowptr[-1]).astype(np.int32)
    ctx().reserve(N, len(colidx), 8, 8, 1 << 17)
    for S in (big, big[:6], big[1:]):
        assert len(S) * d // 2048 > 8192
        rp, ci, v = oracle.induced_csr(N, rowptr, colidx, S)
        out = sg.Csr(len(S), len(S), len(ci), DEV)
        assert _induced(N, rowptr, colidx, S, out) == len(ci)
        assert np.array_equal(out.rowptr.cpu().numpy(), rp) and np.array_equal(out.colidx.cpu().numpy(), ci)
    ctx().status()


def test_plan_of_a_matrix_that_is_filled_again():
    # the plan's counter starts at zero in every call: hub rows, two samples into one matrix, products with and without
    N = 6000
    rng = np.random.default_rng(8)
    deg = np.where(rng.random(N) < 0.05, 3000, 2)
    rowptr = np.concatenate([[0], np.cumsum(deg)])
    colidx = np.concatenate([np.sort(rng.choice(N, d, replace=False)) for d in deg])
    B, E = 3000, len(colidx)
    ctx().reserve(N, E, B, 64, E)
    out = sg.Csr(B, B, E, DEV)
    X = torch.randn(B, 64, device=DEV, generator=torch.Generator(DEV).manual_seed(1))
    for seed in (1, 2, 3):
        S = np.sort(np.random.default_rng(seed).choice(N, B, replace=False))
        nnz = _induced(N, rowptr, colidx, S, out)
        rp, ci, v = oracle.induced_csr(N, rowptr, colidx, S)
        assert nnz == len(ci) and np.array_equal(out.rowptr.cpu().numpy(), rp)
        Y = torch.empty(B, 64, device=DEV)
        sg.sgnn_spmm(ctx(), out, X, Y)
        H = X.cpu().numpy()
        # one rounding for every product and addition, and the weights to TOL_VAL
        bound = (np.diff(rp).max() + 2) * 2.0**-24 + TOL_VAL
        assert np.all(np.abs(Y.cpu().numpy() - oracle.spmm(rp, ci, v, H)) <= bound * oracle.spmm(rp, ci, np.abs(v), np.abs(H)) + 1e-12)


@pytest.mark.parametrize("N,B", [(1200000011, 400000000), (1200000011, 1001), (600000000, 200000001)])
def test_sample_of_a_graph_with_more_candidates_than_the_list_holds(N, B):
    # Exactly B vertices with keys up to one threshold is the whole definition of the sample: the count is taken from the
    # bitmap, and of some vertices the keys.
    c = sg.Context(0)                                    # not the shared one, which would keep room for this size
    c.reserve(N, 1, 1, 1)
    S, W = torch.full((B,), -1, dtype=torch.int32, device=DEV), (N + 63) // 64
    bitmap, rank = torch.full((W,), -1, dtype=torch.int64, device=DEV), torch.empty(W, dtype=torch.int32, device=DEV)
    sg.sgnn_sample_uniform(c, N, B, 5, 3, S, bitmap, rank)
    c.status()
    got = S.cpu().numpy()
    assert np.all(np.diff(got) > 0) and got[0] >= 0 and got[-1] < N
    words = bitmap.cpu().numpy().view(np.uint64)
    assert int(np.bitwise_count(words).sum()) == B
    del S, bitmap, rank
    c.close()
    torch.cuda.empty_cache()
    v = np.r_[np.random.default_rng(1).integers(0, N, 3000), got[np.random.default_rng(2).integers(0, B, 1000)]]
    inside = (words[v >> 6] >> (v & 63).astype(np.uint64)) & np.uint64(1) == 1
    keys = np.array([oracle.vertex_key(5, 3, int(x)) for x in v], np.uint64)
    assert inside[-1000:].all() and keys[inside].max() < keys[~inside].min()
