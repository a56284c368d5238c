"""The sampler of graphs whose keys one workgroup holds (up to 16384 vertices) and the first sizes beyond it."""
import numpy as np
import pytest

import oracle
from gpu_util import bitmap_rank_from_sample, gpu_sample

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
