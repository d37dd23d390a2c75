"""A call that fails in its first tile while thousands of further workgroups of
the same launch are still to start: they leave as a whole, the status says why,
and the next call on the same plan and workspace is unaffected."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

EUNSUPPORTED, ERANGE = -5, -2


def test_oversized_tile_of_many():
    """Over 2^32 payload bytes in the first two of 60 M cells (3,663 tiles)."""
    from paper_2012_06012_amd import mgt
    n, m, w = 1 << 20, 60_000_000, (1 << 31) + 64
    row_ptr = torch.arange(n + 1, device="cuda") * m // n
    col = (torch.arange(m, device="cuda") * 7919 % n).to(torch.int32)
    payload = torch.empty(2 * w, dtype=torch.uint8, device="cuda")
    poff = torch.full((m + 1,), 2 * w, dtype=torch.int64, device="cuda")
    poff[0], poff[1] = 0, w
    a = mgt.DeviceCsr(n, n, row_ptr, col, poff, payload, np.array([0, n], np.int64), 8)
    plan = mgt.plan_for(a)
    ws = mgt.workspace_for(plan, "cuda")
    out, st = mgt.transpose(a, plan=plan, workspace=ws)
    assert int(st.cpu()[0]) == EUNSUPPORTED
    poff[1:m] = w  # the second cell's bytes move to the last one
    out, st = mgt.transpose(a, plan=plan, workspace=ws, out=out)
    assert int(st.cpu()[0]) == 0
    order = torch.sort(col.long(), stable=True)
    rows = torch.searchsorted(row_ptr, order.indices, right=True) - 1
    assert torch.equal(out["t_col"].long(), rows)
    assert torch.equal(out["t_row_ptr"],
                       torch.searchsorted(order.values, torch.arange(n + 1, device="cuda")))
    size = torch.zeros(m, dtype=torch.int64, device="cuda")
    size[0] = size[m - 1] = w
    assert torch.equal(out["t_payload_off"][1:], torch.cumsum(size[order.indices], 0))


@pytest.mark.parametrize("op", [0, 1])
def test_bad_column_of_a_view(op):
    """One column out of range in the first of 9,766 workgroups of cells."""
    from paper_2012_06012_amd import mgt
    n, m = 1 << 16, 20_000_000
    row_ptr = torch.arange(n + 1, device="cuda") * m // n
    col = (torch.arange(m, device="cuda") * 7919 % n).to(torch.int32)
    poff = torch.zeros(m + 1, dtype=torch.int64, device="cuda")
    empty = torch.empty(0, dtype=torch.uint8, device="cuda")
    bounds = np.linspace(0, n, 8).astype(np.int64)
    for bad, want in ((n + 3, ERANGE), (5, 0)):
        col[0] = bad
        out, st = mgt.view_transform(row_ptr, col, poff, empty, n, n, bounds, 8, op, mgt.ROW_VIEW,
                                     validate=True)
        assert int(st.cpu()[0]) == want
    assert int(out["row_ptr"][-1]) == m
