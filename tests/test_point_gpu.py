"""1x1 layers with 8- and 16-bit inputs on their own kernel (chunks of whole channel runs, maps numbered
as one run of pixels): integer-valued inputs against the oracle, bit for bit, between guard bands.
"""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
import paper_1705_10591_amd as dconv

pytestmark = pytest.mark.gpu

TYPES = {"f16": (torch.float16, 2), "bf16": (torch.bfloat16, 2), "i8": (torch.int8, 1)}

# (N, C, H, W, K): runs of 64 and 128 bytes a chunk, one to many chunks, fewer pixels than a tile, tiles
# that end anywhere in an image and span several, filters off multiples of 64; the last four are
# shapes for the 128 x 128, 128 x 64, 64 x 128 and (few channels) 128 x 64 tiles, and an output
# that another kernel takes
SHAPES = [(1, 64, 1, 1, 1), (3, 64, 5, 7, 33), (2, 128, 9, 11, 64), (5, 192, 7, 7, 65), (1, 96, 30, 31, 40),
          (70, 64, 1, 1, 130), (2, 320, 13, 17, 129), (4, 32, 8, 8, 20), (1, 1024, 4, 4, 100),
          (6, 832, 80, 81, 128), (5, 512, 64, 65, 127), (23, 64, 129, 130, 64), (9, 128, 97, 99, 250)]


def lay_out(a, blocked, size):
    """[A, C, h, w] -> [A, h, w, C] or [A, C/cb, h, w, cb]"""
    if not blocked:
        return np.ascontiguousarray(np.moveaxis(a, 1, -1))
    cb = 32 // size
    A, C, h, w = a.shape
    return np.ascontiguousarray(a.reshape(A, C // cb, cb, h, w).transpose(0, 1, 3, 4, 2))


@pytest.mark.parametrize("blocked", [False, True], ids=["last", "blocked"])
@pytest.mark.parametrize("kind", list(TYPES))
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_point_layers_exact(shape, kind, blocked):
    N, C, H, W, K = shape
    dtype, size = TYPES[kind]
    if C * size % 32:
        pytest.skip("no whole channel block")
    x, f = wl.integer_case(9100 + C + K, N, C, H, W, K, 1)
    want = oracle.general(x, f)[0]
    print(f"point {kind} {shape} blocked={blocked}", flush=True)
    xd, fd = (torch.from_numpy(lay_out(a, blocked, size)).to("cuda").to(dtype) for a in (x, f))
    out_type = torch.int32 if kind == "i8" else torch.float32
    fill = -(2**31) if kind == "i8" else float("nan")
    buf = torch.full((want.size + 2048,), fill, device="cuda", dtype=out_type)
    out = buf[1001:1001 + want.size].view(want.shape)
    (dconv.dconv_general_i8 if kind == "i8" else dconv.dconv_general_half)(xd, fd, out=out, blocked=blocked)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy().astype(np.float64), want)
    for band in (buf[:1001], buf[1001 + want.size:]):
        assert bool((band == fill).all()) if kind == "i8" else bool(torch.isnan(band).all())


def test_point_layer_non_finite_pixel_and_filter_stay_where_they_belong():
    x, f = wl.random_case(9200, 3, 64, 9, 10, 70, 1)
    x[1, 5, 3, 4], f[66, 7, 0, 0] = np.nan, np.inf
    xd, fd = (torch.from_numpy(lay_out(a, False, 2)).to("cuda").half() for a in (x, f))
    got = dconv.dconv_general_half(xd, fd).cpu().numpy()
    bad = ~np.isfinite(got)
    want = np.zeros_like(bad)
    want[1, :, 3, 4] = True
    want[:, 66] = True
    assert np.array_equal(bad, want)


@pytest.mark.parametrize("blocked", [False, True], ids=["last", "blocked"])
@pytest.mark.parametrize("kind", ["f16", "bf16"])
@pytest.mark.parametrize("shape", [(5, 192, 7, 7, 65), (2, 320, 13, 17, 129), (6, 832, 80, 81, 128), (5, 512, 64, 65, 127)],
                         ids=lambda s: "x".join(map(str, s)))
def test_point_layers_keep_the_bits_of_the_kernel_for_every_filter_side(shape, kind, blocked):
    """Sums are taken in the same order on both kernels, so rounding is the same too."""
    N, C, H, W, K = shape
    dtype, size = TYPES[kind]
    x, f = wl.random_case(9300 + C + K, N, C, H, W, K, 1)
    print(f"point {kind} {shape} blocked={blocked}", flush=True)
    xd, fd = (torch.from_numpy(lay_out(a, blocked, size)).to("cuda").to(dtype) for a in (x, f))
    got = dconv.dconv_general_half(xd, fd, blocked=blocked)
    for cfg in (0, 1):
        assert torch.equal(got, dconv.dconv_general_half(xd, fd, blocked=blocked, variant=dconv.VARIANT_TILED_CFG0 + cfg)), cfg
