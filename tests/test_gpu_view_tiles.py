"""View operations in the two-launch form (keys as columns, values as rows)
against oracle/views.py: few and many keys (past 1,048,576: the passes), crowded
columns, both views and operations, and 257 partitions (the passes)."""
import numpy as np
import pytest

from oracle import views
from workloads.gen import equal_bounds, from_arrays

from .test_gpu_views import _check, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nnz,parts,law,w_hi", [
    (500, 4097, 1, "uniform", 9), (3000, 100003, 37, "uniform", 33), (9000, 150001, 200, "uniform", 4),
    (9000, 90001, 200, "hot", 12), (20000, 400009, 256, "uniform", 7), (600, 9001, 257, "uniform", 5),
])
@pytest.mark.parametrize("fixed", [False, True])
def test_views(n, nnz, parts, law, w_hi, fixed):
    rng = np.random.default_rng(nnz)
    rp = np.concatenate([[0], np.sort(rng.integers(0, nnz + 1, size=n - 1)), [nnz]])
    col = rng.integers(0, n, nnz)
    if law == "hot":
        col = np.where(rng.random(nnz) < 0.7, n // 2 + rng.integers(0, 3, nnz), col)
        rp = np.concatenate([[0], np.full(n // 2, nnz // 3), np.full(n - n // 2, nnz)])  # two rows
    w = np.full(nnz, w_hi) if fixed else rng.integers(0, w_hi + 1, nnz)
    a = from_arrays(n, n, rp, col.astype(np.int32), w, None, 8, equal_bounds(n, parts))
    x = views.ViewCsr(n, n, views.ROW_VIEW, a.bounds, a.row_ptr, a.col, a.payload_off, a.payload)
    for op, f in ((0, views.local_transpose), (1, views.view_swap)):
        want, perm = f(x)
        h, st = _run(x, op, perm=True, fixed=fixed)
        assert st == 0
        _check(h, want, perm)
        y = want  # a column view
        for op2, f2 in ((0, views.local_transpose), (1, views.view_swap)):
            want2, perm2 = f2(y)
            h2, st2 = _run(y, op2, perm=True, fixed=fixed)
            assert st2 == 0
            _check(h2, want2, perm2)
