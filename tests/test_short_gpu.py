"""Short launches of the general case: small tiles whose reduction the waves of a workgroup share (VARIANT_SHORT, and
AUTO by estimated time).
"""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
import paper_1705_10591_amd as dconv
from helpers import assert_within_bound

pytestmark = pytest.mark.gpu

# (N, C, H, W, K, F): every tile and number of waves; taps that end a step early or not, fewer steps than waves,
# pixels and filters off multiples of a tile, maps smaller than one, many images
SHAPES = [(1, 12, 5, 5, 9, 2), (1, 15, 7, 9, 17, 1), (2, 1, 12, 15, 9, 9), (3, 1, 104, 58, 18, 4),
          (3, 7, 66, 90, 17, 4), (5, 74, 87, 35, 17, 1), (1, 31, 28, 246, 17, 4), (9, 87, 21, 41, 18, 2), (1, 256, 14, 14, 256, 3),
          (8, 50, 30, 30, 90, 3), (64, 33, 7, 7, 65, 3)]
# layers that the library's rule sends elsewhere: three taps, the largest filters
BY_NAME_ONLY = [(7, 3, 41, 58, 18, 1), (2, 40, 20, 17, 40, 11), (1, 3, 40, 40, 33, 32)]
ids = lambda s: "x".join(map(str, s))
SHORT = dconv.VARIANT_SHORT


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


@pytest.mark.parametrize("shape", SHAPES + BY_NAME_ONLY, ids=ids)
def test_within_the_bound_between_guard_bands(shape):
    N, C, H, W, K, F = shape
    print(f"short {shape}", flush=True)
    x, f = wl.random_case(9500 + C + F, N, C, H, W, K, F, "u01", "he")
    fd = dev(f)
    xb = torch.empty(x.size + 1, device="cuda")[1:].view(x.shape)      # images need no alignment beyond a float's
    xb.copy_(dev(x))
    want = (N, K, H - F + 1, W - F + 1)
    buf = torch.full((int(np.prod(want)) + 2048,), float("nan"), device="cuda")
    out = buf[1001:len(buf) - 1047].view(want)
    dconv.dconv_general(xb, fd, out=out, variant=SHORT)
    chosen = dconv.kernel_choice(False, *shape) == SHORT
    assert chosen == (shape not in BY_NAME_ONLY)
    same = [dconv.dconv_general(xb.clone(), fd, noalloc=True, variant=SHORT)] + \
        ([dconv.dconv_general(xb, fd), dconv.dconv_general(xb, fd, noalloc=True)] if chosen else [])
    whole = dconv.dconv_general(xb, fd, variant=dconv.VARIANT_TILED_CFG0 + 3 + dconv.tile_choice(False, *shape))
    tiled = [whole, dconv.dconv_general(xb, fd, variant=dconv.VARIANT_TILED)]
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    acc, mag, _ = oracle.general(x, f)
    assert_within_bound(got, acc, mag, f"short {shape}")
    assert torch.isnan(buf[:1001]).all() and torch.isnan(buf[len(buf) - 1047:]).all()
    assert all(torch.equal(out, o) for o in same)
    assert C * F * F <= 16 or not any(torch.equal(out, o) for o in tiled)
    err = [np.linalg.norm(o.cpu().numpy() - acc) for o in (out, whole)]
    assert C * F * F < 100 or err[0] <= err[1], err
    # one pixel and one weight that are not finite reach their outputs and no other
    at = (N - 1, C - 1, H // 2, W - 2)
    xb[at] = float("nan")
    fd[K - 1, 0, 0, 0] = float("inf")
    marked = dconv.dconv_general(xb, fd, variant=SHORT)
    hit = torch.zeros_like(out, dtype=torch.bool)
    hit[N - 1, :, max(0, at[2] - F + 1):at[2] + 1, max(0, at[3] - F + 1):at[3] + 1] = True
    assert torch.equal(torch.isnan(marked[:, :K - 1]), hit[:, :K - 1]) and torch.equal(marked[:, :K - 1][~hit[:, :K - 1]], out[:, :K - 1][~hit[:, :K - 1]])
    assert not torch.isfinite(marked[:, K - 1]).any()


@pytest.mark.parametrize("shape", SHAPES[::3] + BY_NAME_ONLY, ids=ids)
def test_integer_inputs_are_exact(shape):
    x, f = wl.integer_case(9550, *shape)
    out = dconv.dconv_general(dev(x), dev(f), variant=SHORT)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), oracle.general(x, f)[0].astype(np.float32))


def test_a_captured_call_runs_the_same():
    """No workspace: the replayed graph gives the eager call's bits, with other work between replays."""
    x, f = wl.random_case(9560, 8, 50, 30, 30, 90, 3, "u01", "he")
    xd, fd = dev(x), dev(f)
    eager = dconv.dconv_general(xd, fd)
    assert torch.equal(eager, dconv.dconv_general(xd, fd, variant=SHORT))
    out = torch.zeros_like(eager)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        dconv.dconv_general(xd, fd, out=out)
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager)
        dconv.dconv_general(xd, fd)
