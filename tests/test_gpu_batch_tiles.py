"""Batches whose items take the two-launch form of mid-size calls (tiles.hip),
alone and beside items that make the passes (too many columns or partitions,
no cells), against the oracle; recorded batches; workspaces that only the
passes fit."""
import numpy as np
import pytest
import torch

import oracle
from workloads import gen
from workloads.gen import from_arrays

from .common import assert_matches_oracle, host, to_device

pytestmark = pytest.mark.gpu


def _small(seed, n, deg, w, parts=1, ow=8):
    return gen.random_small(seed, n_rows=n, n_cols=n, deg_mean=deg, w_lo=0, w_hi=w, parts=parts,
                            offset_width=ow)


def _wide(seed, n_cols):  # more columns than one level of buckets holds
    rng = np.random.default_rng(seed)
    return from_arrays(50, n_cols, np.linspace(0, 4000, 51).astype(np.int64),
                       rng.integers(0, n_cols, 4000).astype(np.int32), rng.integers(0, 9, 4000), None, 8)


def _mixed():
    return [_small(1, 3, 2.0, 5), _small(2, 3000, 20.0, 16, parts=7), _wide(3, 3 << 20),
            from_arrays(4, 4, [0] * 5, [], [], None, 8), _small(4, 900, 3.0, 40, parts=300),
            _small(5, 20000, 11.0, 3, parts=64), _small(6, 1, 9.0, 4), _small(7, 700, 60.0, 33, parts=2)]


def _check(mats, outs, st, perm):
    assert (st.cpu().numpy() == 0).all()
    for a, o in zip(mats, outs):
        assert_matches_oracle(a, host(o), check_perm=perm, partitioned=a.n_parts > 1)


@pytest.mark.parametrize("perm", [False, True])
@pytest.mark.parametrize("which", ["mixed", "tiles", "one"])
def test_batches(which, perm):
    from paper_2012_06012_amd import mgt
    mats = _mixed()
    if which == "tiles":
        mats = [a for a in mats if a.n_cols <= 20000 and a.n_parts < 300 and a.nnz]
    elif which == "one":
        mats = mats[1:2]
    outs, st, plan, ws = mgt.batch_transpose([to_device(a) for a in mats], perm=perm)
    _check(mats, outs, st, perm)


def test_many_items():
    """More items than one search round of a workgroup (512)."""
    from paper_2012_06012_amd import mgt
    mats = [_small(100 + i, 5 + i % 40, 3.0, 7, parts=1 + i % 3) for i in range(700)]
    outs, st, _, _ = mgt.batch_transpose([to_device(a) for a in mats])
    _check(mats, outs, st, False)


def test_workspace_of_the_passes(monkeypatch):
    """A workspace sized for the passes alone is accepted and gives the same."""
    from paper_2012_06012_amd import mgt
    mats = [_small(10 + i, 2000 + 100 * i, 12.0, 2) for i in range(4)]
    devs = [to_device(a) for a in mats]
    plan = mgt.batch_plan_for(devs)
    outs = [mgt.alloc_outputs(d) for d in devs]
    entries, keep = mgt.batch_entries(devs, outs)
    items = mgt.make_items(entries)
    both = mgt.mgt_batch_workspace(plan, items)  # at least what the passes take
    monkeypatch.setenv("MGT_NO_TILES", "1")
    passes = mgt.mgt_batch_workspace(plan, items)
    monkeypatch.delenv("MGT_NO_TILES")
    st = torch.empty(len(mats), dtype=torch.int32, device="cuda")
    assert both >= passes
    for need in {both, passes}:
        for o in outs:
            for v in o.values():
                if v is not None:
                    v.fill_(3)
        mgt.mgt_batch_submit(plan, items, torch.empty(need, dtype=torch.uint8, device="cuda"), st)
        torch.cuda.synchronize()
        _check(mats, outs, st, False)
    with pytest.raises(mgt.MgtError):
        mgt.mgt_batch_submit(plan, items, torch.empty(256, dtype=torch.uint8, device="cuda"), st)
    del keep


def test_replays():
    from paper_2012_06012_amd import mgt
    mats = _mixed()
    devs = [to_device(a) for a in mats]
    g, outs, st, plan, ws = mgt.batch_graph(devs)
    rng = np.random.default_rng(0)
    for _ in range(4):
        for a, d in zip(mats, devs):
            a.col[:] = rng.integers(0, a.n_cols, size=a.nnz).astype(np.int32)
            d.col.copy_(torch.from_numpy(a.col.copy()))
        for o in outs:
            for v in o.values():
                if v is not None:
                    v.fill_(7)
        st.fill_(9)
        g.launch()
        torch.cuda.synchronize()
        _check(mats, outs, st, False)
