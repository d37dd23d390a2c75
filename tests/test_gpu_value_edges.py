"""Value-list conversions where their kernels change form: runs that end in the
same 64-cell word, in the next one or many words on, chunks of 1,024 words,
rows and cells that are empty in long stretches, and expansions whose
workgroups (2,048 values) walk or search their cells. Against oracle/values.py."""
import numpy as np
import pytest
import torch

from oracle import values
from workloads.gen import from_arrays

from .common import to_device

pytestmark = pytest.mark.gpu


def _np(t):
    return t.cpu().numpy()


def _runs(rng, n, kind):
    """Columns of n cells in runs of the given lengths."""
    if kind == "one":
        return np.zeros(n, np.int32)
    lens = {"short": [1, 2, 3], "word": [63, 64, 65, 1], "long": [1, 7, 700, 20000]}[kind]
    out = np.repeat(np.arange(n, dtype=np.int32) % 997, rng.choice(lens, size=n))[:n]
    return out


@pytest.mark.parametrize("n", [1, 63, 64, 65, 255, 257, 65535, 65536, 65537, 200003])
@pytest.mark.parametrize("kind,ow", [("one", 8), ("short", 4), ("word", 8), ("long", 4)])
def test_coalesce_runs(n, kind, ow):
    from paper_2012_06012_amd import mgt
    rng = np.random.default_rng(n)
    col = _runs(rng, n, kind)
    # rows: one, or many with long stretches of empty ones at both ends
    for cuts in ([], np.sort(rng.integers(0, n + 1, size=min(n, 300)))):
        rp = np.concatenate([np.zeros(1 + 500 * (len(cuts) > 0), np.int64), cuts,
                             np.full(1 + 3000 * (len(cuts) > 0), n)]).astype(np.int64)
        a = from_arrays(len(rp) - 1, 1000, rp, col, rng.integers(0, 3, size=n), None, ow)
        want = values.coalesce(a.row_ptr, a.col, a.payload_off)
        out, m = mgt.coalesce(to_device(a))
        assert m == want.col.shape[0]
        for k in ("row_ptr", "col", "payload_off", "counts"):
            assert np.array_equal(_np(out[k]).astype(np.int64), getattr(want, k)), k


@pytest.mark.parametrize("nnz,hi,w,ow", [
    (1, 1, 4, 8), (1, 5000, 8, 8), (2047, 1, 4, 4), (2048, 1, 12, 8), (2049, 1, 1, 4),
    (30000, 9, 8, 8),
    (400000, "sparse", 8, 8),     # over 16,384 cells per 2,048 values: searched
    (60000, "gaps", 4, 4),        # both in one call
])
def test_expand_ranges(nnz, hi, w, ow):
    from paper_2012_06012_amd import mgt
    rng = np.random.default_rng(nnz)
    if hi == "sparse":
        cnt = (rng.random(nnz) < 0.01).astype(np.int64)
    elif hi == "gaps":
        cnt = rng.integers(0, 4, size=nnz)
        cnt[5000:40000] = 0
    else:
        cnt = np.full(nnz, hi) if nnz < 3 else rng.integers(0, hi + 1, size=nnz)
    n = 100
    rp = np.concatenate([[0], np.sort(rng.integers(0, nnz + 1, size=n - 1)), [nnz]])
    a = from_arrays(n, 500, rp, rng.integers(0, 500, size=nnz).astype(np.int32), cnt * w, None, ow)
    out, st = mgt.expand(to_device(a), w)
    want = values.expand(a.row_ptr, a.col, a.payload_off, w)
    assert int(st.cpu()[0]) == 0
    for k in ("row_ptr", "col", "payload_off"):
        assert np.array_equal(_np(out[k]).astype(np.int64), getattr(want, k)), k


@pytest.mark.parametrize("at", [0, 1, 4095, 69999])
def test_expand_checks_every_offset(at):
    from paper_2012_06012_amd import mgt
    cnt = np.full(70000, 8)
    cnt[at] = 6
    cnt[(at + 1) % 70000] = 10 if at < 69999 else 8
    if at == 69999:
        cnt[0] = 10
    a = from_arrays(1, 3, [0, 70000], np.zeros(70000, np.int32), cnt, None, 8)
    out, st = mgt.expand(to_device(a), 8)
    assert int(st.cpu()[0]) == mgt.ERANGE
