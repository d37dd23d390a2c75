"""Transfer matrices counted beside the tile sort and added up in the merge, at
the edges of their split: one and several workgroups per source partition, the
last share, a partition holding every cell, the most partitions; a failed device
check leaves them zero."""
import numpy as np
import pytest

import oracle
from workloads.gen import equal_bounds, from_arrays

from .common import assert_matches_oracle, gpu_transpose, host, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _no_direct(monkeypatch):
    monkeypatch.setenv("MGT_NO_DIRECT", "1")  # small sizes take this form too


def _matrix(n, nnz, bounds, seed, crowded=False):
    rng = np.random.default_rng(seed)
    cuts = np.sort(rng.integers(0, nnz + 1, size=n - 1))
    if crowded:  # every cell in one source partition
        cuts[:] = np.where(np.arange(1, n) < bounds[2], 0, nnz)
    rp = np.concatenate([[0], cuts, [nnz]])
    col = rng.integers(0, n, nnz).astype(np.int32)
    return from_arrays(n, n, rp, col, rng.integers(0, 9, nnz), None, 8, bounds)


@pytest.mark.parametrize("parts,nnz", [
    (1, 4095), (1, 4096), (1, 8193), (3, 12287), (3, 12288), (3, 24577),
    (37, 600011), (255, 300007), (256, 1048575), (256, 1048577),
])
@pytest.mark.parametrize("crowded", [False, True])
def test_shares(parts, nnz, crowded):
    a = _matrix(1500, nnz, equal_bounds(1500, parts), nnz, crowded and parts > 2)
    h, st = gpu_transpose(a, partitioned=True, perm=False, validate=bool(nnz & 1))
    assert st == 0
    assert_matches_oracle(a, h, partitioned=True)


@pytest.mark.parametrize("nnz", [25000, 25001])  # the last direct partitioned size, the first past it
def test_edge_of_the_direct_form(nnz, monkeypatch):
    monkeypatch.delenv("MGT_NO_DIRECT")
    a = _matrix(1500, nnz, equal_bounds(1500, 13), nnz)
    h, st = gpu_transpose(a, partitioned=True, perm=True)
    assert st == 0
    assert_matches_oracle(a, h, partitioned=True)


def test_failed_check_leaves_zero():
    from paper_2012_06012_amd import mgt
    a = _matrix(900, 50021, equal_bounds(900, 7), 5)
    d = to_device(a)
    plan = mgt.plan_for(d, mgt.VALIDATE)
    ws = mgt.workspace_for(plan, d.col.device)
    out = mgt.alloc_outputs(d, partitioned=True)
    for bad in (False, True, False):  # the same plan and workspace in between
        good = int(a.col[777])
        d.col[777] = a.n_cols if bad else good
        out["xfer_cells"].fill_(-3)
        out["xfer_bytes"].fill_(-3)
        _, st = mgt.transpose(d, plan=plan, workspace=ws, out=out, partitioned=True, validate=True)
        assert int(st.cpu()[0]) == (mgt.ERANGE if bad else mgt.OK)
        h, pc = host(out), oracle.partition_counts(a)
        for k in ("xfer_cells", "xfer_bytes"):
            assert np.array_equal(h[k], np.zeros_like(h[k]) if bad else getattr(pc, k)), k
