"""Layers of a few tiles, each shared by many workgroups whose sums a second kernel adds (one image of a
deep layer): the tiled kernel (VARIANT_TILED) picks this by size.  Against the oracle, integer inputs bit for bit between
guard bands, the entry point that allocates nothing, and under graph capture.
"""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import workloads as wl
import paper_1705_10591_amd as dconv
from helpers import assert_within_bound

pytestmark = pytest.mark.gpu
TILED = dconv.VARIANT_TILED

# (N, C, H, W, K, F): the three tile shapes, tiles shared unevenly, a channel count that leaves one
# channel a chunk, row groups, filters off multiples of 32, two column strips, 1x1 filters
SHAPES = [(1, 256, 14, 14, 256, 3), (1, 96, 20, 20, 32, 3), (2, 64, 30, 30, 64, 3), (1, 48, 40, 44, 100, 5), (1, 37, 14, 14, 70, 3),
          (1, 16, 30, 31, 33, 7), (1, 8, 40, 41, 64, 11), (1, 6, 30, 30, 20, 13), (1, 256, 14, 14, 256, 1), (3, 32, 28, 28, 64, 4),
          (2, 128, 28, 28, 128, 3), (1, 128, 5, 150, 40, 3)]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_parts_added_by_a_second_kernel(shape):
    N, C, H, W, K, F = shape
    print(f"general {shape}", flush=True)
    x, f = wl.random_case(9500 + C + F, *shape)
    acc, mag, _ = oracle.general(x, f)
    xd, fd = dev(x), dev(f)
    got = dconv.dconv_general(xd, fd, variant=TILED)
    whole = dconv.dconv_general(xd, fd, variant=dconv.VARIANT_TILED_CFG0 + 3 + dconv.tile_choice(False, *shape))
    again, static = dconv.dconv_general(xd, fd, variant=TILED), dconv.dconv_general(xd, fd, variant=TILED, noalloc=True)
    torch.cuda.synchronize()
    assert not torch.equal(got, whole), "the tiles are expected to be shared here"
    assert torch.equal(got, again) and torch.equal(got, static)
    assert_within_bound(got.cpu().numpy(), acc, mag, f"sum of parts {shape}")
    xi, fi = wl.integer_case(9600 + C + F, *shape)
    want = oracle.general(xi, fi)[0].astype(np.float32)
    buf = torch.full((want.size + 2048,), float("nan"), device="cuda")
    out = buf[1001:1001 + want.size].view(want.shape)
    dconv.dconv_general(dev(xi), dev(fi), out=out, variant=TILED)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), want)
    assert torch.isnan(buf[:1001]).all() and torch.isnan(buf[1001 + want.size:]).all()


def kernel_nodes(graph):
    """Kernels that a captured graph holds."""
    hip, n = ctypes.CDLL("libamdhip64.so.7"), ctypes.c_size_t()
    raw = ctypes.c_void_p(graph.raw_cuda_graph())
    assert hip.hipGraphGetNodes(raw, None, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("noalloc", [False, True])
def test_both_kernels_are_captured(noalloc):
    shapes = SHAPES
    cases = [tuple(map(dev, wl.random_case(9700 + i, *s))) for i, s in enumerate(shapes)]
    outs = [torch.empty(N, K, H - F + 1, W - F + 1, device="cuda") for (N, C, H, W, K, F) in shapes]
    s, g = torch.cuda.Stream(), torch.cuda.CUDAGraph(keep_graph=True)

    def enqueue():
        for (x, f), o in zip(cases, outs):
            dconv.dconv_general(x, f, out=o, variant=TILED, noalloc=noalloc)

    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        enqueue()                          # (its workspace exists from here on)
    s.synchronize()
    eager = [o.clone() for o in outs]
    print("capturing", flush=True)
    with torch.cuda.graph(g, stream=s):
        enqueue()
    assert kernel_nodes(g) == 2 * len(shapes), "a second kernel is expected in every call"
    g.instantiate()
    for rep in range(3):
        for o in outs:
            o.fill_(float("nan"))
        other = dconv.dconv_general(*cases[0], variant=TILED)
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(o, e) for o, e in zip(outs, eager)), f"replay {rep}"
        assert torch.equal(other, eager[0])
