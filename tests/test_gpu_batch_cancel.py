"""An item that fails in a batch cancels the others (MGT_ECANCELED), whichever
form each of them takes: here one of over 2^32 payload bytes in two cells, which
makes the passes and gives MGT_EUNSUPPORTED, beside items of the two-launch form
and one of too many columns for it."""
import numpy as np
import pytest
import torch

from workloads import gen
from workloads.gen import from_arrays

from .common import assert_matches_oracle, host, to_device

pytestmark = pytest.mark.gpu

EUNSUPPORTED, ECANCELED = -5, -6


def _small(seed, n, parts=1):
    return gen.random_small(seed, n_rows=n, n_cols=n, deg_mean=9.0, w_lo=0, w_hi=9, parts=parts)


def _oversized():
    from paper_2012_06012_amd import mgt
    w = (1 << 31) + 64  # of each of two cells
    i64 = lambda x: torch.tensor(x, dtype=torch.int64, device="cuda")  # noqa: E731
    return mgt.DeviceCsr(2, 2, i64([0, 1, 2]), torch.tensor([1, 0], dtype=torch.int32, device="cuda"),
                         i64([0, w, 2 * w]), torch.empty(2 * w, dtype=torch.uint8, device="cuda"),
                         np.array([0, 2], np.int64), 8)


@pytest.mark.parametrize("recorded", [False, True], ids=["submit", "graph"])
@pytest.mark.parametrize("at", [0, 2], ids=["first", "last"])
def test_failing_item_cancels_the_others(at, recorded):
    from paper_2012_06012_amd import mgt
    mats = [to_device(_small(1, 900)), to_device(_small(2, 3000, parts=7))]
    mats.insert(at, _oversized())
    if recorded:
        g, outs, st, plan, ws = mgt.batch_graph(mats)
        for _ in range(2):
            st.fill_(9)
            g.launch()
    else:
        outs, st, plan, ws = mgt.batch_transpose(mats)
    got = st.cpu().numpy()
    assert got[at] == EUNSUPPORTED
    assert all(got[i] == ECANCELED for i in range(3) if i != at)


def test_next_batch_on_the_same_workspace_runs():
    """The failure is that batch's own: the next one starts clean."""
    from paper_2012_06012_amd import mgt
    wide = from_arrays(40, 3 << 20, np.linspace(0, 2000, 41).astype(np.int64),
                       (np.arange(2000) * 1499 % (3 << 20)).astype(np.int32),
                       np.arange(2000) % 9, None, 8)
    small = [_small(3, 900), _small(4, 2000, parts=5), wide]
    devs = [to_device(a) for a in small]
    bad = _oversized()
    plan = mgt.mgt_batch_plan(4, 1 << 24, 1 << 24, 1 << 24, 64, 1 << 24, 1 << 24, 8)
    ws = torch.empty(8 << 30, dtype=torch.uint8, device="cuda")
    for mats, want in ((devs + [bad], [ECANCELED] * 3 + [EUNSUPPORTED]), (devs, [0] * 3)):
        outs, st, _, _ = mgt.batch_transpose(mats, plan=plan, workspace=ws)
        assert list(st.cpu().numpy()) == want
    for a, o in zip(small, outs):
        assert_matches_oracle(a, host(o), check_perm=False, partitioned=a.n_parts > 1)
