"""Row starts of mgt_coalesce, which a wave ORs together per 64-cell word: rows
of one cell (64 starts in a word), rows that start in every lane of a word or
one word each, empty rows between and around them, a last partial wave of
rows, an end on a word's boundary. Against oracle/values.py."""
import numpy as np
import pytest

from oracle import values
from workloads.gen import from_arrays

from .common import to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_rows", [1, 63, 64, 65, 129, 4097])
@pytest.mark.parametrize("deg", ["one", "two", "word", "mixed", "gaps"])
def test_row_starts(n_rows, deg):
    from paper_2012_06012_amd import mgt
    rng = np.random.default_rng(n_rows)
    d = {"one": np.ones(n_rows, np.int64), "two": np.full(n_rows, 2), "word": np.full(n_rows, 64),
         "mixed": rng.integers(0, 130, n_rows),
         "gaps": np.where(rng.random(n_rows) < 0.9, 0, rng.integers(1, 4, n_rows))}[deg]
    rp = np.concatenate([[0], np.cumsum(d)])
    nnz = int(rp[-1])
    # one column only: every output cell is a row start
    a = from_arrays(n_rows, 3, rp, np.full(nnz, 2, np.int32), np.full(nnz, 1), None, 8)
    want = values.coalesce(a.row_ptr, a.col, a.payload_off)
    out, m = mgt.coalesce(to_device(a))
    assert m == want.col.shape[0]
    for k in ("row_ptr", "col", "payload_off", "counts"):
        assert np.array_equal(out[k].cpu().numpy().astype(np.int64), getattr(want, k)), k
