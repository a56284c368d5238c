"""Tiles of the induced-matrix passes: rows that start and end on tile edges, row tables at and over their size,
runs of empty rows, hub rows over several tiles - against the CPU oracle, bit-exact on indices."""
import numpy as np
import pytest
import torch

import oracle
import paper_2604_02651_amd as sg
from gpu_util import DEV, TOL_VAL, ctx, gpu_sample

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
