"""mgt_symmetrize where its fill changes form: 2,048 cells of S per workgroup,
rows shorter and longer than that, long stretches of empty rows, payload runs
packed in LDS (up to 32 bytes a cell) and copied lane by lane, both triangles.
Against oracle/symmetric.py."""
import numpy as np
import pytest

from workloads.gen import from_arrays

from .test_gpu_symmetric import _compare

pytestmark = pytest.mark.gpu


def _triangle(n, nnz, lower, law, w_hi, ow, seed):
    rng = np.random.default_rng(seed)
    if law == "dense rows":
        r = rng.choice([n // 3, n - 1], size=nnz)
    elif law == "gaps":      # all rows in a few narrow bands
        r = (rng.integers(0, 4, nnz) * (n // 4) + rng.integers(0, 9, nnz)) % n
    else:
        r = rng.integers(0, n, nnz)
    c = (rng.random(nnz) * (r + 1)).astype(np.int64)
    if not lower:
        r, c = c, r
    o = np.lexsort((c, r))
    r, c = r[o], c[o]
    rp = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=n))])
    return from_arrays(n, n, rp, c.astype(np.int32), rng.integers(0, w_hi + 1, nnz), None, ow)


@pytest.mark.parametrize("lower", [True, False], ids=["lower", "upper"])
@pytest.mark.parametrize("n,nnz,law,w_hi,ow", [
    (1, 5, "uniform", 3, 8), (300, 1024, "uniform", 32, 4), (300, 1025, "uniform", 33, 8),
    (2500, 20011, "dense rows", 9, 8), (60000, 9001, "gaps", 16, 4), (5000, 60013, "uniform", 90, 8),
    (5000, 60013, "uniform", 0, 8),
    # uneven buckets (from 65,536 stored cells): few, crowded and many columns
    (3, 65536, "uniform", 5, 8), (700, 120011, "dense rows", 9, 4), (40000, 200003, "uniform", 20, 8),
    (900000, 300007, "gaps", 4, 8), (1 << 20, 66000, "uniform", 7, 8),
])
def test_fill_edges(n, nnz, law, w_hi, ow, lower):
    _compare(_triangle(n, nnz, lower, law, w_hi, ow, nnz), lower, validate=True)
