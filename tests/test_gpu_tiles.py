"""Mid-size calls (tiles sorted by bucket, then one workgroup per bucket)
against the oracle and against the same call through the passes
(MGT_NO_TILES=1), at the edges of their forms: the last tile, buckets of one
column and of 512, buckets over what a workgroup holds (a hot column), empty
rows, columns and partitions, payloads in the records (up to 4 bytes) and
read from the input at every size and alignment, sizes past a record's field,
perm, device checks, recorded calls."""
import numpy as np
import pytest
import torch

import oracle
from workloads import gen
from workloads.gen import equal_bounds, from_arrays

from .common import assert_matches_oracle, gpu_transpose, host, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _no_direct(monkeypatch):
    monkeypatch.setenv("MGT_NO_DIRECT", "1")  # small sizes take this form too


def _both(a, monkeypatch, partitioned, perm=True, validate=False):
    outs = []
    for off in (False, True):
        if off:
            monkeypatch.setenv("MGT_NO_TILES", "1")
        h, st = gpu_transpose(a, partitioned=partitioned, perm=perm, validate=validate)
        if off:
            monkeypatch.delenv("MGT_NO_TILES")
        assert st == 0
        assert_matches_oracle(a, h, partitioned=partitioned)
        outs.append(h)
    for k, v in outs[0].items():
        assert v is None or np.array_equal(v, outs[1][k]), k


def _matrix(n_rows, n_cols, nnz, law, seed, w_lo, w_hi, ow, parts=1):
    rng = np.random.default_rng(seed)
    if law == "hot":
        col = np.where(rng.random(nnz) < 0.6, n_cols // 2, rng.integers(0, n_cols, nnz))
    elif law == "few":   # a tenth of the columns, at both ends
        col = rng.integers(0, max(1, n_cols // 10), nnz)
        col = np.where(rng.random(nnz) < 0.5, col, n_cols - 1 - col)
    else:
        col = rng.integers(0, n_cols, nnz)
    cuts = np.sort(rng.integers(0, nnz + 1, size=max(0, n_rows - 1)))
    rp = np.concatenate([[0], cuts, [nnz]])
    w = rng.integers(w_lo, w_hi + 1, size=nnz)
    return from_arrays(n_rows, n_cols, rp, col.astype(np.int32), w, None, ow,
                       equal_bounds(n_rows, parts))


@pytest.mark.parametrize("nnz", [1, 63, 64, 65, 1024, 4095, 4096, 4097, 40001, 524288, 524289])
@pytest.mark.parametrize("law,ow,perm", [("uniform", 4, True), ("hot", 8, False), ("few", 8, True)])
def test_cell_counts(nnz, law, ow, perm, monkeypatch):
    _both(_matrix(999, 3000, nnz, law, nnz, 0, 20, ow), monkeypatch, False, perm=perm)


@pytest.mark.parametrize("n_rows,n_cols,law", [
    (1, 2, "uniform"), (3, 1, "uniform"), (70, 511, "few"), (20000, 513, "uniform"),
    (300, 1 << 20, "uniform"), (300, (1 << 20) + 1, "few"), (90000, 40000, "hot"), (5, 3001, "hot"),
])
@pytest.mark.parametrize("w_lo,w_hi", [(0, 7), (9, 20)])
def test_shapes(n_rows, n_cols, law, w_lo, w_hi, monkeypatch):
    _both(_matrix(n_rows, n_cols, 60013, law, n_cols, w_lo, w_hi, 8), monkeypatch, False)


@pytest.mark.parametrize("parts", [1, 2, 37, 256, 257])
@pytest.mark.parametrize("law,w_hi", [("uniform", 23), ("hot", 6)])
def test_partitions(parts, law, w_hi, monkeypatch):
    _both(_matrix(5000, 5000, 200017, law, parts, 0, w_hi, 8, parts), monkeypatch, True)


def test_uneven_partitions_and_empty_rows(monkeypatch):
    b = np.array([0, 0, 3000, 3000, 3001, 7000, 7000], np.int64)
    a = _matrix(7000, 7000, 90001, "uniform", 3, 0, 5, 4)
    rp = np.concatenate([np.zeros(2500, np.int64), a.row_ptr[:1] + 50000, np.full(1500, 50000),
                         np.full(3000, 90001)])
    for m in (from_arrays(7000, 7000, a.row_ptr, a.col, np.diff(a.payload_off), None, 4, b),
              from_arrays(7000, 7000, rp, a.col, np.diff(a.payload_off), None, 8, b)):
        _both(m, monkeypatch, True)


@pytest.mark.parametrize("w_lo,w_hi,pay", [
    (0, 0, gen.PAY_BYTES), (1, 1, gen.PAY_BYTES), (4, 4, gen.PAY_BYTES), (5, 5, gen.PAY_BYTES),
    (8, 8, gen.PAY_BYTES), (0, 8, gen.PAY_BYTES), (0, 16, gen.PAY_BYTES), (9, 17, gen.PAY_BYTES),
    (15, 33, gen.PAY_BYTES), (32, 32, gen.PAY_BYTES), (0, 200, gen.PAY_BYTES),
    (1, 8, gen.PAY_FLOATS)])
@pytest.mark.parametrize("perm", [False, True])
def test_payload_sizes(w_lo, w_hi, pay, perm, monkeypatch):
    a = gen.random_small(w_hi, n_rows=6000, n_cols=5000, deg_mean=9.0, w_lo=w_lo, w_hi=w_hi,
                         pay_law=pay)
    _both(a, monkeypatch, False, perm=perm)


def test_payload_alignment():
    """Sources and destinations at every offset modulo 16, guard bytes around the output kept."""
    from paper_2012_06012_amd import mgt
    a = gen.random_small(1, n_rows=3000, n_cols=2000, deg_mean=8.0, w_lo=0, w_hi=40)
    ref = oracle.transpose(a)
    d = to_device(a)
    plan, n = mgt.plan_for(d), a.payload_bytes
    ws = mgt.workspace_for(plan, d.col.device)
    for s in range(16):
        t = (5 * s + 3) % 16
        src = torch.zeros(n + 64, dtype=torch.uint8, device="cuda")
        src[s:s + n] = d.payload
        dst = torch.full((n + 64,), 0x5A, dtype=torch.uint8, device="cuda")
        out = mgt.alloc_outputs(d)
        out["t_payload"] = dst[t:t + n]
        d.payload = src[s:s + n]
        _, st = mgt.transpose(d, plan=plan, workspace=ws, out=out)
        assert int(st.cpu()[0]) == 0
        h = dst.cpu().numpy()
        assert np.array_equal(h[t:t + n], ref.t_payload)
        assert (h[:t] == 0x5A).all() and (h[t + n:] == 0x5A).all()


@pytest.mark.parametrize("n_cols,nnz,law,ow", [
    (1 << 20, 60013, "uniform", 8),        # the most columns of this form
    ((1 << 20) + 1, 60013, "uniform", 8),  # past it: the passes
    (3 << 20, 200003, "uniform", 4), (8 << 20, 1000, "few", 8), ((8 << 20) + 1, 1000, "few", 8),
    (2 << 20, 70001, "hot", 8),
])
@pytest.mark.parametrize("perm", [False, True])
def test_many_columns(n_cols, nnz, law, ow, perm, monkeypatch):
    _both(_matrix(500, n_cols, nnz, law, nnz, 0, 20, ow), monkeypatch, False, perm=perm)


def test_many_columns_all_crowded(monkeypatch):
    """Every cell in a few neighbouring columns."""
    a = _matrix(500, 3 << 20, 30000, "uniform", 1, 0, 9, 8)
    a.col[:] = 5000 + a.col % 1500
    _both(a, monkeypatch, False)


def test_long_cells_of_many_columns(monkeypatch):
    w = np.full(3000, 3)
    w[[0, 1500, 2999]] = [(1 << 20) - 2, (1 << 20) - 1, (1 << 20) + 5]
    rng = np.random.default_rng(0)
    a = from_arrays(100, 2 << 20, np.linspace(0, 3000, 101).astype(np.int64),
                    rng.integers(0, 2 << 20, 3000).astype(np.int32), w, None, 8)
    _both(a, monkeypatch, False)


def test_sizes_past_the_record_field(monkeypatch):
    w = np.full(3000, 3)
    w[[0, 1500, 2999]] = [(1 << 22) - 2, (1 << 22) - 1, (1 << 22) + 5]
    rng = np.random.default_rng(0)
    a = from_arrays(100, 90, np.linspace(0, 3000, 101).astype(np.int64),
                    rng.integers(0, 90, 3000).astype(np.int32), w, None, 8)
    _both(a, monkeypatch, False)


@pytest.mark.parametrize("w", [0, 4, 8, 28, 33])
def test_fixed_width(w):
    from paper_2012_06012_amd import mgt
    a = gen.random_small(w, n_rows=4000, n_cols=4000, deg_mean=30.0, w_lo=w, w_hi=w, parts=5)
    d = to_device(a, fixed_width=True)
    ref, pc = oracle.transpose(a), oracle.partition_counts(a)
    out = mgt.alloc_outputs(d, perm=True, partitioned=True, payload_off=False)
    _, st = mgt.transpose(d, perm=True, partitioned=True, out=out)
    h = host(out)
    assert int(st.cpu()[0]) == 0
    for k in ("t_row_ptr", "t_col", "t_payload"):
        assert np.array_equal(h[k], getattr(ref, k)), k
    for k in ("xfer_cells", "xfer_bytes", "part_cell_off", "part_byte_off", "sdispls", "rdispls"):
        assert np.array_equal(h[k], getattr(pc, k)), k


def test_device_checks(monkeypatch):
    """Valid data passes; each broken invariant gives MGT_ERANGE, wherever it sits."""
    from paper_2012_06012_amd import mgt
    a = gen.random_small(4, n_rows=9000, n_cols=7000, deg_mean=8.0, w_lo=0, w_hi=9)
    _both(a, monkeypatch, False, validate=True)

    def status(**edit):
        d = to_device(a)
        for name, (at, v) in edit.items():
            getattr(d, name)[at] = v
        _, st = mgt.transpose(d, validate=True)
        return int(st.cpu()[0])

    assert status() == mgt.OK
    nnz, rp, po = a.nnz, a.row_ptr, a.payload_off
    for at in (0, 5000, nnz - 1):
        assert status(col=(at, -1)) == mgt.ERANGE
        assert status(col=(at, a.n_cols)) == mgt.ERANGE
    for at in (0, 4000, 9000):
        assert status(row_ptr=(at, int(rp[at]) + 1 if at in (0, 9000) else int(rp[-1]) + 1)) == mgt.ERANGE
        assert status(row_ptr=(at, -1)) == mgt.ERANGE
    for at in (0, 30000, nnz):
        assert status(payload_off=(at, int(po[-1]) + 1)) == mgt.ERANGE
        assert status(payload_off=(at, -1)) == mgt.ERANGE


@pytest.mark.parametrize("partitioned", [False, True])
def test_replays(partitioned):
    from paper_2012_06012_amd import mgt
    a = gen.random_small(6, n_rows=5000, n_cols=5000, deg_mean=40.0, w_lo=0, w_hi=19, parts=7)
    d = to_device(a)
    g, out, st = mgt.transpose_graph(d, perm=True, partitioned=partitioned)
    rng = np.random.default_rng(0)
    for _ in range(4):
        col = rng.integers(0, a.n_cols, size=a.nnz).astype(np.int32)
        d.col.copy_(torch.from_numpy(col))
        a.col[:] = col
        for v in out.values():
            if v is not None:
                v.fill_(7)
        st.fill_(5)
        g.launch()
        h = host(out)
        assert int(st.cpu()[0]) == 0
        assert_matches_oracle(a, h, partitioned=partitioned)


def test_largest(monkeypatch):
    """The last size of this form and the first past it."""
    for nnz in (2048 * 4096, 2048 * 4096 + 1):
        a = _matrix(300000, 400000, nnz, "uniform", 1, 0, 3, 8)
        h, st = gpu_transpose(a, perm=False)
        assert st == 0
        assert_matches_oracle(a, h)
