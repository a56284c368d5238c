"""The sampler of graphs whose keys one workgroup holds (up to 16384 vertices), and of those (up to 4194304) whose threshold every
workgroup of the emit pass selects for itself."""
import numpy as np
import pytest

import oracle
import paper_2604_02651_amd as sg
from gpu_util import bitmap_rank_from_sample, ctx, fail_next_launch, gpu_sample

pytestmark = pytest.mark.gpu


# whole and ragged last words, pairs and rounds of 2048 vertices; one vertex, all of them and all but one
@pytest.mark.parametrize("N", [1, 2, 3, 63, 64, 65, 127, 2047, 2048, 2049, 8191, 16383, 16384, 16385, 20001])
@pytest.mark.parametrize("part", ["one", "some", "but one", "all"])
def test_small_sample_matches_oracle(N, part):
    B = {"one": 1, "some": (N + 2) // 3, "but one": max(N - 1, 1), "all": N}[part]
    for step in (0, 2**33 + 1):
        S, bitmap, rank = gpu_sample(N, B, 5, step)
        S_ref = oracle.sample_uniform(N, B, 5, step)
        assert np.array_equal(S.cpu().numpy(), S_ref)
        words, rk = bitmap_rank_from_sample(N, S_ref)
        assert np.array_equal(bitmap.cpu().numpy(), words) and np.array_equal(rank.cpu().numpy(), rk)


# a word, two or more a wavefront; the last dense sample that selects in the emit pass and the first with a launch of its own for it,
# the sparse one (another list) between two dense ones
@pytest.mark.parametrize("N,B", [(65537, 65536), (300001, 100), (524289, 200000), (1048575, 400000), (1048577, 500000),
                                 (4194304, 2097152), (4194304, 4096), (4194304, 2097153), (4194305, 2097152)])
def test_threshold_in_the_emit_pass(N, B):
    for step in (1, 2):
        S, bitmap, rank = gpu_sample(N, B, 9, step)
        S_ref = oracle.sample_uniform(N, B, 9, step)
        assert np.array_equal(S.cpu().numpy(), S_ref)
        words, rk = bitmap_rank_from_sample(N, S_ref)
        assert np.array_equal(bitmap.cpu().numpy(), words) and np.array_equal(rank.cpu().numpy(), rk)


# one pass over the keys: a window of one bin and of two, the first and the last vertices, a ragged last word, several tiles of candidates in the
# threshold's part (the largest)
@pytest.mark.parametrize("N,B", [(1048576 + 63, 1), (1048576, 262144 // 2048), (8388607, 131072), (8388607, 4096 * 17), (100000007, 1000000)])
def test_sparse_sample_in_one_pass_over_the_keys(N, B):
    for step in (3, 4):
        S, bitmap, rank = gpu_sample(N, B, 12, step)
        S_ref = oracle.sample_uniform(N, B, 12, step)
        assert np.array_equal(S.cpu().numpy(), S_ref)
        words, rk = bitmap_rank_from_sample(N, S_ref)
        assert np.array_equal(bitmap.cpu().numpy(), words) and np.array_equal(rank.cpu().numpy(), rk)


# a call that fails behind its first kernel leaves no keys in the histogram, nor candidates, for the next one: dense samples without and with stored
# key prefixes, a launch of its own for the threshold, the sparse form
@pytest.mark.parametrize("N,B", [(20001, 5000), (1048577, 500000), (4194305, 2097152), (1048576 + 63, 100)])
def test_sample_after_a_call_that_failed(N, B):
    S_ref = oracle.sample_uniform(N, B, 3, 2)
    for _ in range(2):
        S, bitmap, rank = gpu_sample(N, B, 3, 1)
        fail_next_launch(lambda: sg.sgnn_sample_uniform(ctx(), N, B, 3, 7, S, bitmap, rank))
        S, bitmap, rank = gpu_sample(N, B, 3, 2)
        assert np.array_equal(S.cpu().numpy(), S_ref)
        words, rk = bitmap_rank_from_sample(N, S_ref)
        assert np.array_equal(bitmap.cpu().numpy(), words) and np.array_equal(rank.cpu().numpy(), rk)
