"""Calls of the two-launch form's sizes with a workspace that only the passes fit:
accepted, the same results, nothing written past it. (Where the form needs more than
the passes: batches of many tiny items, few cells over many partitions.)"""
import numpy as np
import pytest
import torch

from workloads import gen
from workloads.gen import equal_bounds, from_arrays

from .common import assert_matches_oracle, host, to_device

pytestmark = pytest.mark.gpu


def _sizes(query, monkeypatch):
    both = query()
    monkeypatch.setenv("MGT_NO_TILES", "1")
    passes = query()
    monkeypatch.delenv("MGT_NO_TILES")
    assert both > passes
    return both, passes


def _fill(outs):
    for o in outs:
        for v in o.values():
            if v is not None:
                v.fill_(3)


def _workspace(n):
    """n bytes, followed by a page that must stay as it is."""
    base = torch.full((n + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    return base[:n], base[n:]


@pytest.mark.parametrize("parts", [1, 3])
@pytest.mark.parametrize("perm", [False, True])
def test_batches(perm, parts, monkeypatch):
    from paper_2012_06012_amd import mgt
    mats = [gen.random_small(i, n_rows=3 + i % 14, n_cols=3 + i % 14, deg_mean=0.7, w_lo=0, w_hi=2, parts=parts)
            for i in range(600)]
    devs = [to_device(a) for a in mats]
    flags = mgt.EMIT_PERM if perm else 0
    plan = mgt.batch_plan_for(devs, perm)
    outs = [mgt.alloc_outputs(d, perm, parts > 1) for d in devs]
    entries, keep = mgt.batch_entries(devs, outs, perm, flags)
    items = mgt.make_items(entries)
    st = torch.empty(len(mats), dtype=torch.int32, device="cuda")
    sizes = _sizes(lambda: mgt.mgt_batch_workspace(plan, items), monkeypatch)

    def check(run):
        _fill(outs)
        st.fill_(9)
        run()
        torch.cuda.synchronize()
        assert (st.cpu().numpy() == 0).all()
        for a, o in list(zip(mats, outs))[::13]:
            assert_matches_oracle(a, host(o), check_perm=perm, partitioned=parts > 1)

    for need in sizes:
        ws, after = _workspace(need)
        check(lambda: mgt.mgt_batch_submit(plan, items, ws, st))
        g = mgt.mgt_batch_graph_create(plan, items, ws, st)
        for _ in range(3):
            check(g.launch)
        assert bool((after == 0xA5).all())
    with pytest.raises(mgt.MgtError):
        mgt.mgt_batch_submit(plan, items, ws[:sizes[1] - 256], st)
    del keep


@pytest.mark.parametrize("n,m,perm", [(1500, 26_000, False), (600, 60_000, True)])
def test_single_calls(n, m, perm, monkeypatch):
    from paper_2012_06012_amd import mgt
    rng = np.random.default_rng(m)
    rp = np.concatenate([[0], np.sort(rng.integers(0, m + 1, n - 1)), [m]])
    a = from_arrays(n, n, rp, rng.integers(0, n, m).astype(np.int32), rng.integers(0, 5, m), None, 4,
                    equal_bounds(n, 256))
    d = to_device(a)
    flags = mgt.EMIT_PERM if perm else 0
    plan = mgt.plan_for(d, flags)
    sizes = _sizes(lambda: mgt.plan_for(d, flags).workspace_bytes, monkeypatch)
    out = mgt.alloc_outputs(d, perm, True)
    for need in sizes:
        ws, after = _workspace(need)
        _fill([out])
        _, st = mgt.transpose(d, plan=plan, workspace=ws, perm=perm, partitioned=True, out=out)
        assert int(st.cpu()[0]) == 0
        assert_matches_oracle(a, host(out), check_perm=perm, partitioned=True)
        g, out, st = mgt.transpose_graph(d, plan=plan, workspace=ws, perm=perm, partitioned=True, out=out)
        for _ in range(3):
            _fill([out])
            g.launch()
            assert_matches_oracle(a, host(out), check_perm=perm, partitioned=True)
        assert bool((after == 0xA5).all())
