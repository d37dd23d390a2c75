"""Single calls whose one pass would leave buckets over what the finish holds
make two (matrices past the two-launch form: over 256 partitions, 1,024
columns' worth of buckets times many cells), against the oracle; a workspace
that holds one pass only still serves them."""

import numpy as np
import pytest
import torch

from workloads import gen
from workloads.gen import equal_bounds

from .common import assert_matches_oracle, host, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,deg,parts,fixed", [(600, 700.0, 300, False), (700, 600.0, 1, False),
                                               (600, 700.0, 300, True)])
def test_two_passes_for_large_buckets(n, deg, parts, fixed, monkeypatch):
    from paper_2012_06012_amd import mgt
    monkeypatch.setenv("MGT_NO_DIRECT", "1")
    monkeypatch.setenv("MGT_NO_TILES", "1")
    a = gen.random_small(n, n_rows=n, n_cols=n, deg_mean=deg, w_lo=9 if fixed else 0, w_hi=9, parts=parts)
    d = to_device(a, fixed_width=fixed)
    plan = mgt.plan_for(d)
    for part in (False, True):
        out, st = mgt.transpose(d, plan=plan, partitioned=part)
        assert int(st.cpu()[0]) == 0
        h = host(out)
        assert_matches_oracle(a, h, check_perm=False, partitioned=part)


def test_one_pass_workspace(monkeypatch):
    """10 M cells in 60,000 columns: two passes by the rule, one where only that fits."""
    from paper_2012_06012_amd import mgt
    n, nnz = 60000, 9_000_000
    rng = np.random.default_rng(0)
    cuts = np.sort(rng.integers(0, nnz + 1, size=n - 1))
    a = gen.from_arrays(n, n, np.concatenate([[0], cuts, [nnz]]), rng.integers(0, n, nnz).astype(np.int32),
                        np.full(nnz, 2), None, 8, equal_bounds(n, 1))
    d = to_device(a)
    plan = mgt.plan_for(d)
    assert plan.schedule()["passes"] == 2
    outs = []
    for need in (plan.workspace_bytes, nnz * 18 + (64 << 20)):
        out = mgt.alloc_outputs(d)
        ws = torch.empty(need, dtype=torch.uint8, device="cuda")
        _, st = mgt.transpose(d, plan=plan, workspace=ws, out=out)
        assert int(st.cpu()[0]) == 0
        outs.append(host(out))
    assert_matches_oracle(a, outs[0], check_perm=False)
    for k, v in outs[0].items():
        assert v is None or np.array_equal(v, outs[1][k]), k
