"""mgt_symmetrize with the workspace of its transpose's single pass, where the call
would rather make two: accepted, the same S, nothing written past it."""
import pytest
import torch

from .common import to_device
from .test_gpu_symmetric_edges import _triangle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lower", [True, False], ids=["lower", "upper"])
def test_workspace_of_one_pass(lower):
    from paper_2012_06012_amd import mgt
    a = to_device(_triangle(2000, 9_000_000, lower, "uniform", 3, 8, 1))
    n, m = a.n_rows, a.nnz
    plan = mgt.plan_for(a)
    assert len(plan.schedule(False)["bits"]) == 2
    most = mgt.mgt_symmetrize_workspace(plan)
    plan.set_schedule(8, 3, 0)  # one pass
    assert len(plan.schedule(False)["bits"]) == 1
    least = mgt.mgt_symmetrize_workspace(plan)
    plan.set_schedule()
    assert least < most
    e = lambda k, t: torch.full((k,), 7, dtype=t, device="cuda")  # noqa: E731
    st, got = e(1, torch.int32), []
    for need in (most, least):
        base = torch.full((need + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
        out = (e(n + 1, torch.int64), e(2 * m, torch.int32), e(2 * m + 1, torch.int64),
               e(2 * a.payload_bytes, torch.uint8), e(2, torch.int64))
        mgt.mgt_symmetrize(plan, 0 if lower else 1, a.row_ptr, a.col, a.payload_off, a.payload, *out,
                           base[:need], st)
        assert int(st.cpu()[0]) == 0
        assert bool((base[need:] == 0xA5).all())
        got.append(out)
    for x, y in zip(*got):
        assert torch.equal(x, y)
    rp, cells = got[0][0], int(got[0][4][0])
    assert int(rp[-1]) == cells == 2 * m - int((a.col.long() == torch.repeat_interleave(
        torch.arange(n, device="cuda"), a.row_ptr[1:] - a.row_ptr[:-1])).sum())
    with pytest.raises(mgt.MgtError):
        mgt.mgt_symmetrize(plan, 0 if lower else 1, a.row_ptr, a.col, a.payload_off, a.payload, *got[0],
                           base[:least - 256], st)
