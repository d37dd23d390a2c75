"""Device checks of calls with far more rows than cells, in the two-launch form:
every row offset is checked (several per thread in flight; the last share and its
remainders), and no slower than by the passes."""
import numpy as np
import pytest
import torch

from .timing import us_per_call

pytestmark = pytest.mark.gpu


def _few_cells(n, m, ow=8, seed=0):
    from paper_2012_06012_amd import mgt
    g = torch.Generator(device="cuda").manual_seed(seed)
    odt = torch.int64 if ow == 8 else torch.int32
    rows, _ = torch.sort(torch.randint(0, n, (m,), device="cuda", generator=g))
    row_ptr = torch.searchsorted(rows, torch.arange(n + 1, device="cuda")).to(odt)
    col = torch.randint(0, 1000, (m,), device="cuda", generator=g).to(torch.int32)
    poff = (torch.arange(m + 1, device="cuda") * 3).to(odt)
    pay = torch.randint(0, 256, (3 * m,), device="cuda", generator=g, dtype=torch.uint8)
    return rows, mgt.DeviceCsr(n, 1000, row_ptr, col, poff, pay, np.array([0, n], np.int64), ow)


@pytest.mark.parametrize("ow", [4, 8])
@pytest.mark.parametrize("n,m", [(4095, 100), (4096, 2500), (4097, 100), (100_001, 1025), (300_000, 9)])
def test_a_bad_row_offset_anywhere(n, m, ow):
    from paper_2012_06012_amd import mgt
    rows, a = _few_cells(n, m, ow)
    out, st = mgt.transpose(a, validate=True)
    assert int(st.cpu()[0]) == 0
    order = torch.sort(a.col, stable=True).indices
    assert torch.equal(out["t_col"].long(), rows[order])
    rng = np.random.default_rng(n + m)
    last = int(torch.nonzero(a.row_ptr == m)[0])  # the first row past the cells
    for i in {0, 1, 511, 512, 4095, n // 2, last, n - 1, n, *rng.integers(0, n + 1, 6).tolist()}:
        good = int(a.row_ptr[i])
        a.row_ptr[i] = m + 1
        assert int(mgt.transpose(a, validate=True)[1].cpu()[0]) == -2, i
        a.row_ptr[i] = good
    assert int(mgt.transpose(a, validate=True)[1].cpu()[0]) == 0


def test_time_of_many_rows(monkeypatch):
    from paper_2012_06012_amd import mgt
    _, a = _few_cells(1 << 24, 100)
    plan = mgt.plan_for(a, mgt.VALIDATE)
    ws, out = torch.empty(plan.workspace_bytes, dtype=torch.uint8, device="cuda"), mgt.alloc_outputs(a)
    st = torch.empty(1, dtype=torch.int32, device="cuda")

    def call():
        mgt.mgt_transpose(plan, a.row_ptr, a.col, a.payload_off, a.payload, out["t_row_ptr"],
                          out["t_col"], out["t_payload_off"], out["t_payload"], None, ws, st)
    tiles = us_per_call(call)
    monkeypatch.setenv("MGT_NO_TILES", "1")
    passes = us_per_call(call)
    assert tiles < 0.9 * passes, (tiles, passes)
