"""Every kernel of dconv_general that has a name, on the smallest and the oddest shapes: exact with whole numbers between
guard bands, or refused with nothing written.
"""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
import paper_1705_10591_amd as dconv

pytestmark = pytest.mark.gpu

NAMES = ["TILED", "FEW_FILTERS", "SPECIAL_CASE", "SHORT", "FEW_TAPS", "FEW_CHANNELS", "PARTS"]
# (N, C, H, W, K, F) and the kernels that run it: one output, one row and one column of outputs, one filter, one channel and
# sixteen, the most taps and one more, the largest filters
SHAPES = [((1, 1, 1, 1, 1, 1), "TILED FEW_FILTERS SPECIAL_CASE SHORT FEW_TAPS"),
          ((1, 1, 2, 2, 1, 2), "TILED FEW_FILTERS SPECIAL_CASE SHORT FEW_TAPS FEW_CHANNELS PARTS"),
          ((3, 2, 11, 11, 5, 11), "TILED SHORT FEW_CHANNELS"),
          ((1, 3, 4, 301, 17, 4), "TILED SPECIAL_CASE SHORT FEW_CHANNELS PARTS"),
          ((2, 3, 302, 4, 17, 4), "TILED SPECIAL_CASE SHORT FEW_CHANNELS"),
          ((300, 1, 3, 3, 2, 3), "TILED FEW_FILTERS SPECIAL_CASE SHORT FEW_TAPS FEW_CHANNELS"),
          ((70, 5, 5, 6, 65, 5), "TILED SHORT FEW_CHANNELS PARTS"),
          ((2, 3, 19, 18, 70, 11), "TILED SHORT FEW_CHANNELS"),
          ((2, 4, 19, 18, 70, 11), "TILED SHORT"),
          ((2, 16, 9, 40, 7, 2), "TILED FEW_FILTERS SHORT FEW_TAPS FEW_CHANNELS PARTS"),
          ((2, 17, 9, 40, 7, 4), "TILED FEW_FILTERS SHORT FEW_TAPS PARTS"),
          ((2, 2, 9, 40, 113, 1), "TILED SPECIAL_CASE SHORT"),
          ((1, 300, 8, 9, 16, 1), "TILED FEW_FILTERS SHORT FEW_TAPS"),
          ((1, 2, 12, 70, 2, 7), "TILED FEW_FILTERS SHORT FEW_TAPS FEW_CHANNELS PARTS"),
          ((1, 2, 33, 33, 3, 33), "")]


@pytest.mark.parametrize("name", NAMES)
@pytest.mark.parametrize("shape,runs", SHAPES, ids=["x".join(map(str, s)) for s, _ in SHAPES])
def test_exact_or_refused(shape, runs, name):
    print(f"{name} {shape}", flush=True)
    N, C, H, W, K, F = shape
    x, f = wl.integer_case(9990 + C + F, *shape)
    want = oracle.general(x, f)[0].astype(np.float32)
    xd, fd = torch.from_numpy(x).cuda(), torch.from_numpy(f).cuda()
    for noalloc in (False, True):
        buf = torch.full((want.size + 2048,), float("nan"), device="cuda")
        out = buf[1001:1001 + want.size].view(want.shape)
        if name in runs.split():
            dconv.dconv_general(xd, fd, out=out, variant=getattr(dconv, "VARIANT_" + name), noalloc=noalloc)
            torch.cuda.synchronize()
            bad = int((out.cpu().numpy() != want).sum())
            assert bad == 0, f"{bad} of {want.size} outputs"
            assert torch.isnan(buf[:1001]).all() and torch.isnan(buf[1001 + want.size:]).all()
        else:
            with pytest.raises(dconv.DconvError) as e:
                dconv.dconv_general(xd, fd, out=out, variant=getattr(dconv, "VARIANT_" + name), noalloc=noalloc)
            assert e.value.status == dconv.STATUS_UNSUPPORTED
            torch.cuda.synchronize()
            assert torch.isnan(buf).all()
