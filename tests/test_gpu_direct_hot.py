"""Small calls whose cells crowd into few columns, in the one-launch form: a wave
with as many cells as its list holds (384: 6,144 cells in one column) and more,
columns of more and of at most four cells of 64, zero-byte and long cells between;
against the oracle, and no slower than without that form."""
import numpy as np
import pytest
import torch

from workloads.gen import equal_bounds, from_arrays

from .common import assert_matches_oracle, gpu_transpose, to_device
from .timing import us_per_call

pytestmark = pytest.mark.gpu


def _cols(law, m, n, rng):
    u = rng.integers(0, n, m)
    if law == "one":
        return np.full(m, n // 3)
    if law == "half":
        return np.where(rng.random(m) < 0.5, n // 3, u)
    if law == "blocks":       # 15, 16, 17, 4 and 5 cells of a column in a row
        reps = np.tile([15, 16, 17, 4, 5, 1, 64], m // 100 + 1)
        return np.repeat(rng.integers(0, n, reps.size), reps)[:m]
    if law == "five":
        return rng.integers(0, 5, m) * (n // 5)
    if law == "neighbours":   # columns of one workgroup
        return n // 2 + rng.integers(0, 9, m)
    return (float(n) ** rng.random(m)).astype(np.int64) - 1  # "zipf"


def _matrix(law, m, n, w_hi, ow, parts=1, seed=0):
    rng = np.random.default_rng(seed + m)
    rp = np.concatenate([[0], np.sort(rng.integers(0, m + 1, n - 1)), [m]])
    w = rng.integers(0, w_hi + 1, m)
    w[rng.random(m) < 0.1] = 0
    return from_arrays(n, n, rp, _cols(law, m, n, rng).astype(np.int32), w, None, ow, equal_bounds(n, parts))


@pytest.mark.parametrize("law", ["one", "half", "blocks", "five", "neighbours", "zipf"])
@pytest.mark.parametrize("m,n,w_hi,ow", [
    (1000, 300, 9, 8), (1025, 50, 33, 4), (4096, 300, 16, 8), (4097, 20000, 40, 8), (6144, 500, 7, 4),
    (6145, 9000, 9, 8), (20_011, 900, 32, 4), (45_000, 3000, 12, 8),
])
def test_plain(law, m, n, w_hi, ow):
    a = _matrix(law, m, n, w_hi, ow)
    h, st = gpu_transpose(a, perm=True)
    assert st == 0
    assert_matches_oracle(a, h)


@pytest.mark.parametrize("law", ["one", "zipf"])
@pytest.mark.parametrize("m", [4097, 25_000])
def test_partitioned(law, m):
    a = _matrix(law, m, 1200, 20, 8, parts=7)
    h, st = gpu_transpose(a, partitioned=True, perm=True)
    assert st == 0
    assert_matches_oracle(a, h, partitioned=True)


@pytest.mark.parametrize("m,n_cols", [(20_000, 1), (45_000, 2), (45_000, 11)])
def test_few_columns(m, n_cols):
    rng = np.random.default_rng(m + n_cols)
    rp = np.concatenate([[0], np.sort(rng.integers(0, m + 1, 999)), [m]])
    a = from_arrays(1000, n_cols, rp, rng.integers(0, n_cols, m).astype(np.int32), rng.integers(0, 9, m), None, 8)
    h, st = gpu_transpose(a, perm=True)
    assert st == 0
    assert_matches_oracle(a, h)


@pytest.mark.parametrize("law", ["one", "half", "five", "zipf"])
@pytest.mark.parametrize("m", [5000, 20_000, 45_000])
def test_time(law, m, monkeypatch):
    from paper_2012_06012_amd import mgt
    a = to_device(_matrix(law, m, m // 16, 16, 8))
    plan, o = mgt.plan_for(a), mgt.alloc_outputs(a)
    ws = torch.empty(plan.workspace_bytes, dtype=torch.uint8, device="cuda")

    def call():
        mgt.mgt_transpose(plan, a.row_ptr, a.col, a.payload_off, a.payload, o["t_row_ptr"], o["t_col"],
                          o["t_payload_off"], o["t_payload"], None, ws)
    direct = us_per_call(call)
    monkeypatch.setenv("MGT_NO_DIRECT", "1")
    other = us_per_call(call)
    assert direct < 1.1 * other, (direct, other)
