"""The general case's few-filters kernel stages rows that begin on 16-byte boundaries 16 bytes a lane and all
others 4 bytes a lane.  The aligned image against the oracle, and bit for bit against the same image one
word off its boundary; a NaN reaches the outputs of its own window only.
"""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
import paper_1705_10591_amd as dconv
from helpers import assert_within_bound

pytestmark = pytest.mark.gpu

FEW = dconv.VARIANT_FEW_FILTERS

# (N, C, H, W, K, F): tiles of 256, 128 and 64 columns ending inside, at and one piece beyond a tile; one and two
# channels a trip with an odd channel count; one, two and four rows a band; 6x6 and 7x7 filters, staged
# with 4 bytes a lane from two filters on; the smallest map
SHAPES = [(1, 5, 9, 260, 3, 3), (2, 3, 40, 256, 1, 7), (1, 7, 33, 264, 8, 3), (3, 5, 14, 132, 2, 1), (2, 4, 21, 128, 16, 5),
          (5, 3, 30, 68, 4, 4), (4, 6, 19, 64, 12, 2), (1, 5, 7, 8, 3, 7), (200, 3, 64, 72, 3, 3), (40, 2, 160, 300, 4, 6),
          (40, 2, 160, 300, 2, 3), (6, 5, 40, 100, 13, 7), (9, 3, 33, 60, 6, 7), (2, 3, 50, 204, 3, 6)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_wide_and_narrow_staging(shape):
    N, C, H, W, K, F = shape
    print(f"few filters {shape}", flush=True)
    x, f = wl.random_case(9800 + W + F, *shape)
    fd, xd = torch.from_numpy(f).cuda(), torch.from_numpy(x).cuda()
    off = torch.empty(x.size + 1, device="cuda")[1:].view(x.shape).copy_(xd)
    assert xd.data_ptr() % 16 == 0 and off.data_ptr() % 16 == 4 and W % 4 == 0
    buf = torch.full((N * K * (H - F + 1) * (W - F + 1) + 2048,), float("nan"), device="cuda")
    got = buf[1001:len(buf) - 1047].view(N, K, H - F + 1, W - F + 1)
    dconv.dconv_general(xd, fd, out=got, variant=FEW)
    narrow = dconv.dconv_general(off, fd, variant=FEW)
    at = (N - 1, C - 1, H // 2, W - 2)
    xd[at] = float("nan")
    marked = dconv.dconv_general(xd, fd, variant=FEW)
    torch.cuda.synchronize()
    assert torch.equal(got, narrow)
    assert torch.isnan(buf[:1001]).all() and torch.isnan(buf[len(buf) - 1047:]).all()
    hit = torch.zeros_like(got, dtype=torch.bool)
    hit[N - 1, :, max(0, at[2] - F + 1):at[2] + 1, max(0, at[3] - F + 1):at[3] + 1] = True
    assert torch.equal(torch.isnan(marked), hit) and torch.equal(marked[~hit], got[~hit])
    acc, mag, _ = oracle.general(x, f)
    assert_within_bound(got.cpu().numpy(), acc, mag, f"few filters {shape}")
