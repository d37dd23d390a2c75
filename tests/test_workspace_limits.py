"""Workspace of the largest calls, from the plans alone (no GPU): a call that fits
the device's 288 GB with the workspace of one pass is not asked for more, and what
fits with room to spare makes two passes at most."""
import numpy as np
import pytest

HBM = 288e9


def _plan(n, nnz, w, parts):
    from paper_2012_06012_amd import mgt
    b = np.linspace(0, n, parts + 1).astype(np.int64) if parts > 1 else None
    return mgt.mgt_plan(n, n, nnz, nnz * w, 8, b)


@pytest.mark.parametrize("n,nnz,w,parts", [
    (1 << 18, (1 << 32) - 1, 4, 1), (1 << 18, (1 << 32) - 1, 4, 256), (1 << 18, 1 << 31, 24, 1),
    (1 << 16, (1 << 32) - 1, 0, 1), (1 << 16, (1 << 32) - 1, 4, 1), (1 << 17, 3 << 30, 8, 64),
])
def test_largest_calls_fit_the_device(n, nnz, w, parts):
    arrays = nnz * (4 + 8) * 2 + 2 * nnz * w  # columns, offsets and payload, in and out
    p = _plan(n, nnz, w, parts)
    assert arrays + p.workspace_bytes < 0.9 * HBM
    for partitioned in {False, parts > 1}:
        assert len(p.schedule(partitioned)["bits"]) == 1


@pytest.mark.parametrize("n,nnz,w,parts", [
    (1 << 18, 1 << 27, 28, 256), (1 << 18, 1 << 30, 28, 256), (1 << 18, 1 << 28, 8, 1),
    (1 << 16, 1 << 30, 16, 1), (1 << 18, (1 << 30) + 4097, 4, 7),
])
def test_a_split_call_makes_two_passes_at_most(n, nnz, w, parts):
    p = _plan(n, nnz, w, parts)
    for partitioned in {False, parts > 1}:
        assert len(p.schedule(partitioned)["bits"]) <= 2
