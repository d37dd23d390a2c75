"""The two-launch form at its most columns (2^20: 2,048 buckets of 512) with the
cells in few neighbouring ones: on both sides of a bucket's edge, in the first and
last bucket, past what a bucket holds at once (4,608), with long cells between."""
import numpy as np
import pytest

from workloads.gen import from_arrays

from .common import assert_matches_oracle, gpu_transpose

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("first,span", [(5000, 1500), (511, 2), (0, 3), ((1 << 20) - 700, 700), (1 << 19, 1)])
@pytest.mark.parametrize("perm", [False, True])
def test_neighbouring_columns(first, span, perm, monkeypatch):
    monkeypatch.setenv("MGT_NO_DIRECT", "1")
    m, rng = 60_013, np.random.default_rng(first + span)
    w = rng.integers(0, 9, m)
    w[[0, m // 2, m - 1]] = [(1 << 22) - 1, 100, (1 << 22) + 5]  # either side of the record's size field
    rp = np.concatenate([[0], np.sort(rng.integers(0, m + 1, 499)), [m]])
    a = from_arrays(500, 1 << 20, rp, (first + rng.integers(0, span, m)).astype(np.int32), w, None, 8)
    h, st = gpu_transpose(a, perm=perm, validate=span == 3)
    assert st == 0
    assert_matches_oracle(a, h, check_perm=perm)
