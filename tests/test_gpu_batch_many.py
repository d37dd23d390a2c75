"""Batches of hundreds of tiny items, where the host's work per item counts: the
submit takes no longer with the two-launch form than by the passes."""
import numpy as np
import pytest
import torch

from workloads.gen import from_arrays

from .common import assert_matches_oracle, host, to_device
from .timing import us_per_call

pytestmark = pytest.mark.gpu


def test_time_of_a_submit():
    from paper_2012_06012_amd import mgt
    rng = np.random.default_rng(3)
    items, mats = [], []
    for _ in range(512):
        rp = np.concatenate([[0], np.sort(rng.integers(0, 11, 15)), [10]])
        mats.append(from_arrays(16, 16, rp, rng.integers(0, 16, 10).astype(np.int32),
                                rng.integers(0, 9, 10), None, 8))
    devs = [to_device(a) for a in mats]
    plan, outs = mgt.batch_plan_for(devs), [mgt.alloc_outputs(d) for d in devs]
    entries, keep = mgt.batch_entries(devs, outs)
    items = mgt.make_items(entries)
    ws = torch.empty(mgt.mgt_batch_workspace(plan, items), dtype=torch.uint8, device="cuda")
    st = torch.empty(512, dtype=torch.int32, device="cuda")
    both = us_per_call(lambda: mgt.mgt_batch_submit(plan, items, ws, st))
    assert (st.cpu().numpy() == 0).all()
    for a, o in list(zip(mats, outs))[::37]:
        assert_matches_oracle(a, host(o), check_perm=False)
    plan.set_schedule(8, -1, 0)  # keeps the passes
    ws = torch.empty(mgt.mgt_batch_workspace(plan, items), dtype=torch.uint8, device="cuda")
    passes = us_per_call(lambda: mgt.mgt_batch_submit(plan, items, ws, st))
    assert both < 1.25 * passes, (both, passes)
    del keep
