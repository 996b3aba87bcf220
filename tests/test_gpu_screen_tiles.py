"""Screening counts at the edges of the kernel's tiles and regions against
the oracle's definitions: 32-word masks, 2048-word tiles, one, four and
sixteen waves per stream, each way of counting gaps, streams that start at
any word address, and runs without a hit across masks, tiles and regions."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import screens
from paper_1501_07701_amd import mtgp, workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    mtgp.lib()
    return t


@pytest.mark.parametrize("span_log2,bins", [(27, 64), (29, 16), (30, 5), (30, 33), (31, 16),
                                            (32, 2)])
@pytest.mark.parametrize("count", [3, 31, 32, 33, 64, 2047, 2049, 4096, 4097, 8192, 8225, 30001,
                                   32769, 98305])
def test_counts_at_mask_tile_and_region_edges(torch, count, span_log2, bins):
    print("case screen count=%d span=2^%d bins=%d" % (count, span_log2, bins), flush=True)
    n = 5
    x = (workloads.splitmix64(np.arange(n * count, dtype=np.uint64), 0x71E + count)
         >> np.uint64(32)).astype(np.uint32).reshape(n, count)
    lo = 0 if span_log2 >= 31 else 0x1234567
    hi = min(lo + (1 << span_log2), 0xFFFFFFFF)
    miss, hit = (0xFFFFFFFF, lo)
    x[1, count // 5:count // 5 + count // 2] = miss     # a gap over tiles and regions
    x[2, :] = miss                                       # no hit, or only the ends
    x[2, [0, count - 1]] = hit
    x[3, :] = hit
    x[4, count // 3:count // 3 + 40] = 0x7FFF            # weight 15, then 17, 14 and 18
    x[4, :3] = (0x1FFFF, 0x3FFF, 0x3FFFF)[:count]
    buf = torch.zeros(n * count + 1, dtype=torch.int32, device="cuda")
    d_x = buf[1:]                                        # not 8-byte aligned
    d_x.copy_(torch.from_numpy(x.view(np.int32).reshape(-1)))
    d_c = torch.full((n * (bins + 9),), -1, dtype=torch.int64, device="cuda")
    mtgp.screen(d_x, n, count, lo, hi, bins, d_c)
    got = d_c.cpu().numpy().view(np.uint64).reshape(n, bins + 9)
    for k in range(n):
        assert np.array_equal(got[k, :bins], screens.gap_counts(x[k], lo, hi, bins)), k
        assert np.array_equal(got[k, bins:].reshape(3, 3), screens.hwd_counts(x[k])), k
