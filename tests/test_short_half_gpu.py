"""Short launches with 8- and 16-bit inputs: small tiles whose reduction the waves of a workgroup share (VARIANT_SHORT,
and AUTO by estimated time).
"""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
import paper_1705_10591_amd as dconv
from helpers import assert_within_bound
from test_point_gpu import TYPES, lay_out

pytestmark = pytest.mark.gpu

# (N, C, H, W, K, F): every tile; an odd number of 32-byte units, fewer steps than waves, pixels and filters off
# multiples of a tile, maps smaller than one, one output, many images, 1x1 filters of odd runs (the last: 8 bits only)
SHAPES = [(1, 32, 5, 5, 9, 2), (1, 96, 7, 9, 17, 1), (3, 32, 3, 3, 1, 3), (1, 256, 14, 14, 256, 3), (2, 160, 9, 20, 33, 5),
          (13, 96, 10, 12, 65, 3), (64, 32, 7, 7, 70, 7), (4, 64, 28, 28, 130, 4), (5, 224, 23, 31, 50, 2),
          (15, 32, 43, 19, 34, 4),
          (25, 192, 25, 24, 34, 2), (13, 384, 40, 17, 66, 2), (6, 480, 36, 36, 135, 2), (18, 128, 37, 44, 16, 7)]
# layers that AUTO runs on the tiled kernel, with channels last and blocked
ELSEWHERE = {False: [(25, 192, 25, 24, 34, 2)], True: []}
ids = lambda s: "x".join(map(str, s))
SHORT = dconv.VARIANT_SHORT


def run(kind, *args, **kw):
    return (dconv.dconv_general_i8 if kind == "i8" else dconv.dconv_general_half)(*args, **kw)


def device(a, kind, blocked):
    dtype, size = TYPES[kind]
    return torch.from_numpy(lay_out(a, blocked, size)).to("cuda").to(dtype)


@pytest.mark.parametrize("blocked", [False, True], ids=["last", "blocked"])
@pytest.mark.parametrize("kind", list(TYPES))
@pytest.mark.parametrize("shape", SHAPES, ids=ids)
def test_integer_inputs_are_exact_between_guard_bands(shape, kind, blocked):
    print(f"short {kind} {shape} blocked={blocked}", flush=True)
    x, f = wl.integer_case(9700 + shape[1] + shape[4], *shape)
    want = oracle.general(x, f)[0]
    fill = -(2**31) if kind == "i8" else float("nan")
    buf = torch.full((want.size + 2048,), fill, device="cuda", dtype=torch.int32 if kind == "i8" else torch.float32)
    out = buf[1001:1001 + want.size].view(want.shape)
    run(kind, device(x, kind, blocked), device(f, kind, blocked), out=out, blocked=blocked, variant=SHORT)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy().astype(np.float64), want)
    for band in (buf[:1001], buf[1001 + want.size:]):
        assert bool((band == fill).all()) if kind == "i8" else bool(torch.isnan(band).all())


@pytest.mark.parametrize("blocked", [False, True], ids=["last", "blocked"])
@pytest.mark.parametrize("kind", ["f16", "bf16"])
@pytest.mark.parametrize("shape", SHAPES[3:-1], ids=ids)
def test_within_the_bound_and_no_further_off_than_the_tiled_kernel(shape, kind, blocked):
    N, C, H, W, K, F = shape
    print(f"short {kind} {shape} blocked={blocked}", flush=True)
    x, f = wl.random_case(9800 + C + F, *shape, "u01", "he")
    xr, fr = wl.to_16bit(x, kind)[0], wl.to_16bit(f, kind)[0]
    xd, fd = device(xr, kind, blocked), device(fr, kind, blocked)
    out, tiled, auto = (run(kind, xd, fd, blocked=blocked, variant=v) for v in (SHORT, dconv.VARIANT_TILED, dconv.VARIANT_AUTO))
    torch.cuda.synchronize()
    acc, mag, _ = oracle.general(xr, fr)
    assert_within_bound(out.cpu().numpy(), acc, mag, f"short {kind} {shape}")
    assert not torch.equal(out, tiled)
    assert torch.equal(auto, tiled if shape in ELSEWHERE[blocked] else out), "small tiles are expected to run here, or not to"
    err = [np.linalg.norm(o.cpu().numpy() - acc) for o in (out, tiled)]
    print(f"  errors {err}", flush=True)
    assert err[0] <= err[1], err
    # one pixel and one weight that are not finite reach their outputs and no other (weights next to the last
    # unit of a filter are the next filter's)
    xr[N - 1, C - 1, H // 2, W - 2], fr[K - 1, 0, 0, 0] = np.nan, np.inf
    marked = run(kind, device(xr, kind, blocked), device(fr, kind, blocked), blocked=blocked, variant=SHORT)
    hit = torch.zeros_like(out, dtype=torch.bool)
    hit[N - 1, :, max(0, H // 2 - F + 1):H // 2 + 1, max(0, W - 2 - F + 1):W - 1] = True
    assert torch.equal(torch.isnan(marked[:, :K - 1]), hit[:, :K - 1])
    assert torch.equal(marked[:, :K - 1][~hit[:, :K - 1]], out[:, :K - 1][~hit[:, :K - 1]])
    assert not torch.isfinite(marked[:, K - 1]).any()


def test_images_and_filters_off_sixteen_bytes_run_elsewhere():
    x, f = wl.integer_case(9900, 1, 64, 9, 9, 20, 3)
    want = oracle.general(x, f)[0]
    xd, fd = device(x, "f16", False), device(f, "f16", False)
    shifted = torch.empty(xd.numel() + 1, device="cuda", dtype=torch.float16)[1:].view(xd.shape)
    shifted.copy_(xd)
    assert np.array_equal(dconv.dconv_general_half(shifted, fd).cpu().numpy().astype(np.float64), want)


@pytest.mark.parametrize("kind", list(TYPES))
def test_a_captured_call_runs_the_same(kind):
    """The replayed graph gives the eager call's bits, with other work between replays."""
    x, f = wl.integer_case(9910, 13, 96, 10, 12, 65, 3)
    xd, fd = device(x, kind, False), device(f, kind, False)
    eager = run(kind, xd, fd)
    assert torch.equal(eager, run(kind, xd, fd, variant=SHORT))
    out = torch.zeros_like(eager)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run(kind, xd, fd, out=out)
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager)
        run(kind, xd, fd)


def test_what_small_tiles_cannot_run_is_refused_by_name():
    x, f = wl.integer_case(9920, 1, 8, 9, 9, 20, 3)            # (channels that are no whole 32 bytes)
    with pytest.raises(dconv.DconvError) as e:
        run("f16", device(x, "f16", False), device(f, "f16", False), variant=SHORT)
    assert e.value.status == dconv.STATUS_UNSUPPORTED
