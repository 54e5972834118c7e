"""Few channels on the fp16 matrix cores, each value as two fp16 parts under a scale of its block (AUTO, by
size).  The shapes are small ones that the library's rule sends there: a call that ran on this kernel differs
in its last bits from the fp32 kernel of the shape's tile and is closer to the exact sums.
"""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
import paper_1705_10591_amd as dconv
from helpers import assert_within_bound

pytestmark = pytest.mark.gpu

# (N, C, H, W, K, F): one to four blocks of sixteen filters (each off a multiple of sixteen), one and two
# filter blocks; filters that stay in LDS beside a small and a large image block, or pass through it; pixels
# numbered through the batch and image by image; strips whose last quads are cut, tiles over three images
SHAPES = [(1, 6, 193, 311, 9, 4), (2, 6, 189, 159, 9, 4), (5, 15, 180, 101, 9, 2), (7, 5, 50, 134, 17, 10), (8, 7, 81, 71, 17, 8),
          (9, 3, 154, 90, 18, 6), (5, 1, 208, 134, 19, 11), (4, 6, 72, 394, 17, 4), (4, 3, 78, 135, 35, 10), (8, 10, 44, 143, 33, 5),
          (7, 2, 89, 205, 33, 5), (8, 3, 165, 83, 34, 5), (5, 15, 53, 373, 35, 2), (4, 6, 52, 278, 49, 6), (9, 1, 62, 123, 97, 8),
          (9, 15, 149, 46, 100, 2), (47, 3, 98, 41, 32, 11), (1, 1, 409, 724, 130, 9)]
ids = lambda s: "x".join(map(str, s))


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def call(x, f, variant=dconv.VARIANT_AUTO, noalloc=False):
    print(f"general {tuple(x.shape)} K,F={f.shape[0]},{f.shape[-1]} variant={variant:#x}", flush=True)
    out = dconv.dconv_general(dev(x), dev(f), variant=variant, noalloc=noalloc)
    torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("shape", SHAPES, ids=ids)
def test_within_the_bound_and_closer_than_the_fp32_kernel(shape):
    N, C, H, W, K, F = shape
    x, f = wl.random_case(9000 + C + F, N, C, H, W, K, F)
    acc, mag, _ = oracle.general(x, f)
    # (the general kernel on whole tiles of the shape the library names; one image of one channel: its own kernel)
    tile = dconv.tile_choice(False, *shape)
    got, fp32 = call(x, f), call(x, f, dconv.VARIANT_TILED_CFG0 + 3 + tile if tile >= 0 else dconv.VARIANT_SPECIAL_CASE)
    assert not np.array_equal(got, call(x, f, dconv.VARIANT_TILED))
    assert not np.array_equal(got, fp32), "the kernel of few channels is expected to run here"
    assert_within_bound(got, acc, mag, f"few channels {shape}")
    err = np.linalg.norm(got - acc), np.linalg.norm(fp32 - acc)
    assert err[0] <= err[1], err
    assert np.array_equal(call(x, f), got) and np.array_equal(call(x, f, noalloc=True), got)


@pytest.mark.parametrize("shape", SHAPES, ids=ids)
def test_integer_inputs_exact_between_guard_bands(shape):
    N, C, H, W, K, F = shape
    x, f = wl.integer_case(9100 + C + F, N, C, H, W, K, F)
    want = oracle.general(x, f)[0].astype(np.float32)
    buf = torch.full((want.size + 2048,), float("nan"), device="cuda")
    out = buf[1001:1001 + want.size].view(want.shape)
    xb = torch.empty(x.size + 1, device="cuda")[1:].view(x.shape)      # images need no alignment beyond a float's
    xb.copy_(dev(x))
    print(f"integers {shape}", flush=True)
    dconv.dconv_general(xb, dev(f), out=out)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), want)
    assert torch.isnan(buf[:1001]).all() and torch.isnan(buf[1001 + want.size:]).all()


@pytest.mark.parametrize("shape", [(8, 10, 44, 143, 33, 5), (9, 1, 62, 123, 97, 8)], ids=ids)
def test_values_that_two_parts_cannot_carry(shape):
    """Infinities and NaN, values next to the largest and the smallest float, blocks whose values span more than
    two fp16 parts under one scale do: what fp32 gives."""
    N, C, H, W, K, F = shape
    x, f = wl.random_case(9200 + F, N, C, H, W, K, F)
    rng = np.random.default_rng(F)
    xb, fb = x.copy(), f.copy()
    for bad in (np.nan, np.inf, -np.inf, 3.4e38, -3.39e38):
        xb[rng.integers(N), rng.integers(C), rng.integers(H), rng.integers(W)] = bad
    fb[K - 1, C - 1, 0, 0], fb[5, 0, F - 1, 0] = np.inf, np.nan
    with np.errstate(all="ignore"):
        acc, mag, _ = oracle.general(xb, fb)
        got = call(xb, fb)
    fits = np.abs(acc) < 3.3e38
    assert np.array_equal(np.isnan(got), np.isnan(acc))
    assert np.array_equal(got[np.isinf(acc)], acc[np.isinf(acc)])
    assert fits.any() and np.all(np.abs(got[fits] - acc[fits]) <= 1e-5 * mag[fits])
    half = np.where(np.arange(W) < W // 2, 1.0, 2.0 ** -60).astype(np.float32)
    spread = np.exp2(rng.integers(-40, 40, size=x.shape)).astype(np.float32)
    per_filter = np.exp2(rng.integers(-60, 60, size=(K, 1, 1, 1))).astype(np.float32)
    for xs, fs in ((x * np.float32(2.0 ** -120), f), (x * np.float32(2.0 ** -128), f * np.float32(2.0 ** 20)), (x * half, f), (x * spread, f),
                   (x, f * per_filter), (x * spread, f * per_filter), (x * np.float32(2.0 ** 100), f), (np.zeros_like(x), f)):
        acc, mag, _ = oracle.general(xs, fs)
        got = call(xs, fs)
        # (a reference sum of subnormal products may be off by half the smallest float a term)
        assert np.all(np.abs(got - acc) <= 1e-5 * mag + C * F * F * 2.0 ** -150)


@pytest.mark.parametrize("shape", [(8, 10, 44, 143, 33, 5), (9, 1, 62, 123, 97, 8)], ids=ids)
def test_filters_of_few_weights_are_summed_in_fp32(shape):
    """Filters of one weight beside full ones give their products rounded once, filters of twelve weights what
    twelve roundings give, and a pixel that is not finite reaches them through their zero weights too."""
    N, C, H, W, K, F = shape
    rng = np.random.default_rng(9300 + F)
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    f = rng.standard_normal((K, C, F, F)).astype(np.float32)
    one = [(k, rng.integers(C), rng.integers(F), rng.integers(F), np.float32(rng.standard_normal())) for k in range(0, K, 4)]
    for k, c, i, j, w in one:
        f[k] = 0
        f[k, c, i, j] = w
    f[2].reshape(-1)[rng.permutation(C * F * F)[12:]] = 0
    got = call(x, f)
    for k, c, i, j, w in one:
        assert np.array_equal(got[:, k], x[:, c, i:i + H - F + 1, j:j + W - F + 1] * w)
    acc, mag, _ = oracle.general(x, f)
    assert np.all(np.abs(got[:, 2] - acc[:, 2]) <= 12 * 2.0 ** -24 * mag[:, 2])
    assert_within_bound(got, acc, mag, f"few weights {shape}")
    x[0, 0, H // 2, W // 2] = np.inf
    with np.errstate(all="ignore"):
        acc, _, _ = oracle.general(x, f)
    assert np.array_equal(np.isnan(call(x, f)), np.isnan(acc))
