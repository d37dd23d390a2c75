"""Transfer matrices of source partitions that share the cells unevenly: shares of
4,096 cells cut at the partitions, a workgroup per piece. Partitions that
end on a share, inside one, many within one, one over all; single calls and
batches against the oracle; the time of a crowded call against an even one's."""
import numpy as np
import pytest
import torch

from workloads.gen import equal_bounds, from_arrays

from .common import assert_matches_oracle, gpu_transpose, host, to_device
from .timing import us_per_call

pytestmark = pytest.mark.gpu


def _matrix(cells, seed, ow=8):
    """Source partition s holds cells[s] cells in its 5 rows."""
    rng = np.random.default_rng(seed)
    R, n = len(cells), 5 * len(cells)
    rp = [0]
    for m in cells:
        rp += sorted((rp[-1] + rng.integers(0, m + 1, size=4)).tolist()) + [rp[-1] + m]
    rp = np.array(rp)
    assert len(rp) == n + 1
    m = int(rp[-1])
    return from_arrays(n, n, rp, rng.integers(0, n, m).astype(np.int32), rng.integers(0, 6, m), None,
                       ow, equal_bounds(n, R))


def _laws():
    one = [3] * 255
    one.insert(200, 300_000)
    return {
        "on the shares": [4096, 8192, 0, 0, 4096, 40960], "one past": [4097, 8191, 1, 0, 4095, 40961],
        "empty ends": [0, 0, 50_000, 0, 0], "one crowded": one, "tiny ones": [200] * 256,
        "one source": [60_001], "last": [0] * 63 + [200_000], "ramp": [37 * i for i in range(64)],
        "large": [2_097_152, 5, 0, 40_000], "largest": [5_000_000, 0, 1, 700_000],
    }


@pytest.fixture
def no_direct(monkeypatch):
    monkeypatch.setenv("MGT_NO_DIRECT", "1")


@pytest.mark.parametrize("law", list(_laws()))
def test_single(law, no_direct):
    a = _matrix(_laws()[law], 7, 4 if law == "ramp" else 8)
    for validate in (False, True):
        h, st = gpu_transpose(a, partitioned=True, perm=False, validate=validate)
        assert st == 0
        assert_matches_oracle(a, h, partitioned=True)


def test_batch():
    from paper_2012_06012_amd import mgt
    laws = _laws()
    del laws["one source"]
    mats = [_matrix(cells, i) for i, cells in enumerate(laws.values())]
    mats.insert(2, from_arrays(9, 9, [0] * 5 + [3000] * 5, np.arange(3000) % 9, np.arange(3000) % 3, None, 8))
    outs, st, _, _ = mgt.batch_transpose([to_device(a) for a in mats])
    assert (st.cpu().numpy() == 0).all()
    for a, o in zip(mats, outs):
        assert_matches_oracle(a, host(o), check_perm=False, partitioned=a.n_parts > 1)


def _device(m, crowded, seed=0):
    from paper_2012_06012_amd import mgt
    n = m // 16
    g = torch.Generator(device="cuda").manual_seed(seed)
    rows, _ = torch.sort(torch.randint(n - n // 64 if crowded else 0, n, (m,), device="cuda", generator=g))
    row_ptr = torch.searchsorted(rows, torch.arange(n + 1, device="cuda"))
    col = torch.randint(0, n, (m,), device="cuda", generator=g).to(torch.int32)
    poff = torch.arange(m + 1, device="cuda") * 8
    return mgt.DeviceCsr(n, n, row_ptr, col, poff, torch.zeros(8 * m, dtype=torch.uint8, device="cuda"),
                         equal_bounds(n, 64), 8)


def _time_single(a):
    from paper_2012_06012_amd import mgt
    plan, o = mgt.plan_for(a), mgt.alloc_outputs(a, partitioned=True)
    ws = torch.empty(plan.workspace_bytes, dtype=torch.uint8, device="cuda")
    return us_per_call(lambda: mgt.mgt_transpose_partitioned(
        plan, a.row_ptr, a.col, a.payload_off, a.payload, o["t_row_ptr"], o["t_col"],
        o["t_payload_off"], o["t_payload"], None, o["xfer_cells"], o["xfer_bytes"],
        o["part_cell_off"], o["part_byte_off"], o["sdispls"], o["rdispls"], ws))


def _time_batch(mats):
    from paper_2012_06012_amd import mgt
    plan = mgt.batch_plan_for(mats)
    entries, keep = mgt.batch_entries(mats, [mgt.alloc_outputs(a, partitioned=True) for a in mats])
    items = mgt.make_items(entries)
    ws = torch.empty(mgt.mgt_batch_workspace(plan, items), dtype=torch.uint8, device="cuda")
    return us_per_call(lambda: mgt.mgt_batch_submit(plan, items, ws))


def test_time_single():
    even, crowded = (_time_single(_device(1_000_000, c)) for c in (False, True))
    assert crowded < 2.5 * even, (crowded, even)


def test_time_batch():
    even, crowded = (_time_batch([_device(300_000, c, i) for i in range(8)]) for c in (False, True))
    assert crowded < 2 * even, (crowded, even)
