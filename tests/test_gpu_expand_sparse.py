"""mgt_expand of few values over many empty cells (one value per thread) and of
long lists with long runs of empty cells between (over 16,384 between a
workgroup's first value and its last: searched by way of samples). Against
torch; no slower than as many cells of one value each."""
import numpy as np
import pytest
import torch

from .timing import us_per_call

pytestmark = pytest.mark.gpu


def _sizes(law, m):
    z = np.zeros(m, np.int64)
    if law == "every 100th":
        z[::100] = 1
    elif law == "every 9th":
        z[::9] = 1
    elif law == "ends":
        z[0] = z[-1] = m
    elif law == "ends and one":
        z[0], z[m // 2], z[-1] = 3000, 1, 1500
    elif law == "two gaps":  # over 2^19 values in all
        z[0], z[m // 2], z[-1] = 300_000, 7, 300_005
    elif law == "last":
        z[-1] = 5
    elif law == "ones":
        z[:] = 1
    return z


def _device(law, m, w, ow):
    odt = torch.int32 if ow == 4 else torch.int64
    off = np.concatenate([[0], np.cumsum(_sizes(law, m) * w)])
    rp = torch.tensor([0, m // 3, m], dtype=odt, device="cuda")
    col = torch.randint(0, 1 << 30, (m,), device="cuda").to(torch.int32)
    return rp, col, torch.from_numpy(off).to("cuda").to(odt)


def _call(rp, col, off, w, ow):
    from paper_2012_06012_amd import mgt
    total = int(off[-1])
    nv = total // w
    e = lambda n, t: torch.empty(n, dtype=t, device="cuda")  # noqa: E731
    out = e(3, rp.dtype), e(nv, torch.int32), e(nv + 1, rp.dtype), e(1, torch.int32)
    return out, lambda: mgt.mgt_expand(2, col.numel(), total, ow, w, rp, col, off, *out)


@pytest.mark.parametrize("ow", [4, 8])
@pytest.mark.parametrize("law,m,w", [
    ("every 100th", 400_000, 8), ("every 100th", 1_000_003, 12), ("every 9th", 300_001, 4),
    ("ends", 16_384, 8), ("ends", 16_386, 8), ("ends", 100_003, 4), ("ends", 300_000, 8),
    ("two gaps", 600_000, 8), ("two gaps", 600_003, 1), ("two gaps", 16_386, 8), ("ends and one", 40_000, 8),
    ("ends and one", 3_000_001, 1), ("ends", 300_000, 1 << 21),
    ("two gaps", 300_000, 3 << 20), ("last", 50_000, 8), ("last", 17_000_001, 3),
])
def test_values(law, m, w, ow):
    if ow == 4 and int(_sizes(law, m).sum()) * w >= 1 << 31:
        pytest.skip("offsets past 4 bytes")
    rp, col, off = _device(law, m, w, ow)
    out, call = _call(rp, col, off, w, ow)
    call()
    cell = torch.repeat_interleave(torch.arange(m, device="cuda"), (off[1:] - off[:-1]).long() // w)
    assert int(out[3].cpu()[0]) == 0
    assert torch.equal(out[1], col[cell])
    assert torch.equal(out[2].long(), torch.arange(cell.numel() + 1, device="cuda") * w)
    assert torch.equal(out[0], off[rp.long()] // w)


@pytest.mark.parametrize("law,m", [("every 100th", 5_000_000), ("every 9th", 300_000), ("ends", 200_000)])
def test_time(law, m):
    ones = us_per_call(_call(*_device("ones", m, 8, 8), 8, 8)[1])
    far = us_per_call(_call(*_device(law, m, 8, 8), 8, 8)[1])
    assert far < 1.2 * ones, (far, ones)
