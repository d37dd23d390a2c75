"""mgt_symmetrize of graphs with long stretches of vertices without an edge: a
workgroup of its fill walks about 16,384 rows between two of its cells at most and
searches the rows of its cells beyond that, so no input makes one workgroup walk the
rest alone. Values against oracle/symmetric.py; the call takes little longer
than the transpose inside it."""
import numpy as np
import pytest
import torch

from workloads.gen import from_arrays

from .test_gpu_symmetric import _compare
from .timing import us_per_call

pytestmark = pytest.mark.gpu


def _ends(n, nnz, band, lower, w_hi, ow, seed):
    """All edges among the first `band` and among the last `band` vertices."""
    rng = np.random.default_rng(seed)
    base = np.where(rng.random(nnz) < 0.5, 0, n - band)
    r, c = base + rng.integers(0, band, nnz), base + rng.integers(0, band, nnz)
    r, c = (np.maximum(r, c), np.minimum(r, c)) if lower else (np.minimum(r, c), np.maximum(r, c))
    o = np.lexsort((c, r))
    r, c = r[o], c[o]
    rp = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=n))])
    return from_arrays(n, n, rp, c.astype(np.int32), rng.integers(0, w_hi + 1, nnz), None, ow)


@pytest.mark.parametrize("lower", [True, False], ids=["lower", "upper"])
@pytest.mark.parametrize("n,nnz,band,ow", [
    # just below, at and past the stretch that is walked; single cells on both sides
    (16384 + 600, 5000, 300, 8), (16384 + 2, 2, 1, 4), (16385 + 1, 7, 1, 8), (16386 + 1, 7, 1, 8),
    (16384 + 256 + 40, 3000, 20, 4), (16384 + 513, 9, 1, 8), (3_000_017, 50_000, 900, 8), (40_000, 2500, 3, 8),
])
def test_values_across_a_gap(n, nnz, band, ow, lower):
    _compare(_ends(n, nnz, band, lower, 20, ow, nnz + n), lower, validate=True)


def test_time_of_a_long_gap():
    """2^24 vertices of which 8,000 have edges. With one workgroup walking the
    gap the call took twice the transpose of the stored triangle."""
    from paper_2012_06012_amd import mgt
    from .common import to_device
    a = to_device(_ends(1 << 24, 60_000, 4000, True, 8, 8, 5))
    n, m = a.n_rows, a.nnz
    plan = mgt.plan_for(a)
    e = lambda k, t: torch.empty(k, dtype=t, device="cuda")  # noqa: E731
    ws, tws = e(mgt.mgt_symmetrize_workspace(plan), torch.uint8), e(plan.workspace_bytes, torch.uint8)
    out = (e(n + 1, torch.int64), e(2 * m, torch.int32), e(2 * m + 1, torch.int64),
           e(2 * a.payload_bytes, torch.uint8), e(2, torch.int64))
    t = mgt.alloc_outputs(a)
    st = e(1, torch.int32)
    args = (a.row_ptr, a.col, a.payload_off, a.payload)
    transpose = us_per_call(lambda: mgt.mgt_transpose(
        plan, *args, t["t_row_ptr"], t["t_col"], t["t_payload_off"], t["t_payload"], None, tws, st))
    whole = us_per_call(lambda: mgt.mgt_symmetrize(plan, 0, *args, *out, ws, st))
    assert whole < 1.5 * transpose, (whole, transpose)
