"""Small calls (up to 45,000 cells: one launch, no workspace) against the
oracle and against the same call by the other forms (MGT_NO_DIRECT=1), at the
edges of their forms: 64-cell rounds, a wave's list of 256 cells (a hot column
outgrows it), row offsets in LDS (up to 8,191 rows) or searched in memory, 256
columns per workgroup, 256 partitions, every payload copy."""
import numpy as np
import pytest
import torch

import oracle
from workloads import gen
from workloads.gen import equal_bounds, from_arrays

from .common import assert_matches_oracle, gpu_transpose, host, to_device

pytestmark = pytest.mark.gpu

PART_KEYS = ("xfer_cells", "xfer_bytes", "part_cell_off", "part_byte_off", "sdispls", "rdispls")


def _both(a, monkeypatch, partitioned, perm=True):
    """The call run directly and by the other forms: equal, and equal to the oracle's."""
    outs = []
    for off in (False, True):
        if off:
            monkeypatch.setenv("MGT_NO_DIRECT", "1")
        h, st = gpu_transpose(a, partitioned=partitioned, perm=perm)
        if off:
            monkeypatch.delenv("MGT_NO_DIRECT")
        assert st == 0
        assert_matches_oracle(a, h, partitioned=partitioned)
        outs.append(h)
    for k, v in outs[0].items():
        assert v is None or np.array_equal(v, outs[1][k]), k


def _matrix(n_rows, n_cols, nnz, law, seed, w_hi, ow, parts=1):
    rng = np.random.default_rng(seed)
    if law == "hot":        # most cells in one column
        col = np.where(rng.random(nnz) < 0.9, n_cols // 2, rng.integers(0, n_cols, nnz))
    elif law == "ends":     # first and last column only
        col = np.where(rng.random(nnz) < 0.5, 0, n_cols - 1)
    else:
        col = rng.integers(0, n_cols, nnz)
    cuts = np.sort(rng.integers(0, nnz + 1, size=max(0, n_rows - 1)))
    rp = np.concatenate([[0], cuts, [nnz]])
    w = rng.integers(0, w_hi + 1, size=nnz)
    return from_arrays(n_rows, n_cols, rp, col.astype(np.int32), w, None, ow,
                       equal_bounds(n_rows, parts))


@pytest.mark.parametrize("nnz", [1, 2, 63, 64, 65, 255, 256, 257, 1023, 1025, 16385])
@pytest.mark.parametrize("law,ow", [("uniform", 4), ("hot", 8), ("ends", 4)])
def test_cell_counts(nnz, law, ow, monkeypatch):
    _both(_matrix(37, 500, nnz, law, nnz, 9, ow), monkeypatch, False)


@pytest.mark.parametrize("n_rows,n_cols,law", [
    (1, 1, "uniform"), (8190, 300, "uniform"), (8191, 257, "uniform"), (8192, 256, "hot"),
    (40000, 70, "uniform"), (300, 65536, "uniform"), (300, 65535, "ends"), (5, 40000, "hot"),
    (300, 65537, "uniform"),  # too many columns
])
def test_shapes(n_rows, n_cols, law, monkeypatch):
    _both(_matrix(n_rows, n_cols, 30011, law, n_cols, 13, 8), monkeypatch, False)


@pytest.mark.parametrize("nnz", [45000, 45001])  # the last direct size, the first past it
def test_largest(nnz, monkeypatch):
    _both(_matrix(4000, 4000, nnz, "uniform", 1, 33, 8, 9), monkeypatch, True)


@pytest.mark.parametrize("parts", [1, 2, 7, 64, 256, 257])
@pytest.mark.parametrize("law", ["uniform", "hot"])
def test_partitions(parts, law, monkeypatch):
    _both(_matrix(700, 700, 20011, law, parts, 21, 8, parts), monkeypatch, True)


def test_empty_partitions_and_rows(monkeypatch):
    b = np.array([0, 0, 300, 300, 301, 700, 700], np.int64)
    a = _matrix(700, 700, 9001, "uniform", 3, 5, 4)
    a.bounds = b
    _both(a, monkeypatch, True)
    rp = np.concatenate([np.zeros(500, np.int64), np.full(201, 9001)])
    _both(from_arrays(700, 700, rp, a.col, np.diff(a.payload_off), None, 8, b), monkeypatch, True)


@pytest.mark.parametrize("w", [0, 1, 4, 16, 17, 28, 32, 33, 100])
def test_fixed_width(w):
    from paper_2012_06012_amd import mgt
    a = gen.random_small(w, n_rows=900, n_cols=900, deg_mean=9.0, w_lo=w, w_hi=w, parts=5)
    d = to_device(a, fixed_width=True)
    ref, pc = oracle.transpose(a), oracle.partition_counts(a)
    out = mgt.alloc_outputs(d, perm=True, partitioned=True, payload_off=False)
    _, st = mgt.transpose(d, perm=True, partitioned=True, out=out)
    h = host(out)
    assert int(st.cpu()[0]) == 0
    for k in ("t_row_ptr", "t_col", "t_payload"):
        assert np.array_equal(h[k], getattr(ref, k)), k
    for k in PART_KEYS:
        assert np.array_equal(h[k], getattr(pc, k)), k


@pytest.mark.parametrize("w_lo,w_hi,pay", [(0, 3, gen.PAY_BYTES), (0, 16, gen.PAY_BYTES),
                                           (17, 32, gen.PAY_BYTES), (0, 80, gen.PAY_BYTES),
                                           (1, 8, gen.PAY_FLOATS)])
def test_payload_copies(w_lo, w_hi, pay, monkeypatch):
    _both(gen.random_small(w_hi, n_rows=2000, n_cols=1500, deg_mean=8.0, w_lo=w_lo, w_hi=w_hi,
                           pay_law=pay), monkeypatch, False)


@pytest.mark.parametrize("partitioned", [False, True])
def test_replays_and_no_allocation(partitioned):
    """Recorded small calls read their inputs anew; the allocation-free entry gives the same."""
    from paper_2012_06012_amd import mgt
    a = gen.tiny(seed=5)
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
    plan = mgt.plan_for(d, mgt.EMIT_PERM)
    o2 = mgt.alloc_outputs(d, perm=True, partitioned=partitioned)
    args = [o2[k] for k in ("t_row_ptr", "t_col", "t_payload_off", "t_payload", "perm")]
    part = [o2[k] for k in PART_KEYS] if partitioned else [None] * 6
    mgt.mgt_transpose_noalloc(plan, partitioned, d.row_ptr, d.col, d.payload_off, d.payload, *args,
                              *part, st)
    h2 = host(o2)
    for k, v in h2.items():
        assert v is None or np.array_equal(v, h[k]), k


@pytest.mark.parametrize("seed,parts,sort_rows,ow", [(0, 1, True, 8), (1, 4, False, 4), (2, 300, True, 8)])
def test_passes_on_small_inputs(seed, parts, sort_rows, ow, monkeypatch):
    """Small calls through the passes (device checks, set schedules and other sizes take them)."""
    monkeypatch.setenv("MGT_NO_DIRECT", "1")
    monkeypatch.setenv("MGT_NO_TILES", "1")
    a = gen.random_small(seed, n_rows=3000, n_cols=3000, deg_mean=11.0, w_lo=0, w_hi=9,
                         sort_rows=sort_rows, offset_width=ow, parts=parts)
    for partitioned in (False, True):
        h, st = gpu_transpose(a, partitioned=partitioned)
        assert st == 0
        assert_matches_oracle(a, h, partitioned=partitioned)
