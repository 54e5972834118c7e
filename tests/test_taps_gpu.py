"""Few channels on the bf16 matrix cores, each value as the sum of three bf16 parts, reduction over taps
(VARIANT_FEW_CHANNELS, and AUTO where its estimated time is the least).  The shapes are small ones that reach every
instantiation of the kernel, which is called by name.
"""
import threading

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
          (9, 12, 149, 46, 100, 2), (47, 3, 98, 41, 32, 11), (1, 1, 409, 724, 130, 9), (3, 8, 40, 61, 16, 8)]
ids = lambda s: "x".join(map(str, s))
FEW_CHANNELS = dconv.VARIANT_FEW_CHANNELS


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def call(x, f, variant=FEW_CHANNELS, noalloc=False):
    print(f"general {tuple(x.shape)} K,F={f.shape[0]},{f.shape[-1]} variant={variant:#x}", flush=True)
    out = dconv.dconv_general(dev(x), dev(f), variant=variant, noalloc=noalloc)
    torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("shape", SHAPES, ids=ids)
def test_within_the_bound_and_closer_than_the_fp32_kernel(shape):
    N, C, H, W, K, F = shape
    x, f = wl.random_case(9000 + C + F, N, C, H, W, K, F)
    acc, mag, _ = oracle.general(x, f)
    got, fp32 = call(x, f), call(x, f, dconv.VARIANT_TILED)
    assert not np.array_equal(got, fp32)
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
    dconv.dconv_general(xb, dev(f), out=out, variant=FEW_CHANNELS)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), want)
    assert torch.isnan(buf[:1001]).all() and torch.isnan(buf[1001 + want.size:]).all()


@pytest.mark.parametrize("shape", [(8, 10, 44, 143, 33, 5), (9, 1, 62, 123, 97, 8)], ids=ids)
def test_values_that_two_parts_cannot_carry(shape):
    """Infinities and NaN, values next to the largest and the smallest float: what fp32 gives."""
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
def test_only_what_parts_cannot_give_is_formed_again(shape):
    """A tiny pixel that no sum is small enough to feel leaves all bits as they are (no filter is missing from the
    last block of sixteen for nothing), a filter of tiny weights those of the other blocks."""
    N, C, H, W, K, F = shape
    x, f = wl.random_case(9250 + F, N, C, H, W, K, F)
    x[:, 0, ::9, ::11] = 0
    want, y, g = call(x, f), x.copy(), f.copy()
    y[:, 0, ::9, ::11] = 2.0 ** -110
    g[20] *= np.float32(2.0 ** -110)
    assert np.array_equal(call(y, f), want)
    got = call(x, g)
    other = np.arange(K) // 16 != 1
    assert np.array_equal(got[:, other], want[:, other])
    acc, mag, _ = oracle.general(x, g)
    assert np.all(np.abs(got[:, 20] - acc[:, 20]) <= 1e-5 * mag[:, 20] + C * F * F * 2.0 ** -150)


@pytest.mark.parametrize("shape", [(8, 10, 44, 143, 33, 5), (9, 1, 62, 123, 97, 8), (3, 3, 50, 39, 64, 11)], ids=ids)
def test_filters_of_few_weights(shape):
    """Filters of one weight beside full ones give their products rounded once (rows that end off a multiple of
    four included), filters of twelve weights what
    twelve roundings give, and a pixel that is not finite reaches them through their zero weights too."""
    N, C, H, W, K, F = shape
    rng = np.random.default_rng(9300 + F)
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    f = rng.standard_normal((K, C, F, F)).astype(np.float32)
    one = [(k, rng.integers(C), rng.integers(F), rng.integers(F), np.float32(rng.standard_normal())) for k in range(0, K, 4)]
    one[-1] = (one[-1][0], C - 1, F - 1, F - 1, np.float32(2.0 ** -110))      # (its products are no sums that are formed again)
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


@pytest.mark.parametrize("weights", [2, 3, 12])
def test_banks_of_sparse_filters_are_no_further_off_than_on_the_fp32_kernel(weights):
    N, C, H, W, K, F = shape = (3, 3, 80, 90, 48, 7)
    x, f = wl.random_case(9390 + weights, *shape)
    rng = np.random.default_rng(weights)
    for k in range(K):
        f[k].reshape(-1)[rng.permutation(C * F * F)[weights:]] = 0
    acc, mag, _ = oracle.general(x, f)
    got, fp32 = (call(x, f, v) for v in (FEW_CHANNELS, dconv.VARIANT_TILED))
    assert_within_bound(got, acc, mag, f"{weights} weights")
    assert np.linalg.norm(got - acc) <= np.linalg.norm(fp32 - acc)


def test_whole_numbers_are_exact_while_their_sums_are():
    """Products of 24 bits: odd pixels of 12 bits under a weight of 12 bits among small ones, and pixels of 24 bits, one a
    window, under powers of two."""
    N, C, H, W, K, F = 8, 10, 44, 143, 33, 5
    rng = np.random.default_rng(9400)
    x = (2 * rng.integers(1024, 2048, (N, C, H, W)) + 1).astype(np.float32)
    f = rng.choice([-1.0, 0.0, 1.0], (K, C, F, F)).astype(np.float32)
    f.reshape(K, -1)[np.arange(K), rng.integers(0, C * F * F, K)] = rng.choice([-2049.0, 2049.0, 2051.0], K)
    y = np.zeros((N, C, H, W), np.float32)
    y[:, 3, 2::F, 1::F] = 2 * rng.integers(1 << 22, 1 << 23, y[:, 3, 2::F, 1::F].shape) + 1
    g = rng.choice([-4.0, -1.0, 0.5, 1.0, 2.0], (K, C, F, F)).astype(np.float32)
    for xs, fs in ((x, f), (y, g)):
        want = oracle.general(xs, fs)[0]
        assert np.array_equal(want, want.astype(np.float32))
        assert np.array_equal(call(xs, fs), want.astype(np.float32))


# few taps, where a sum has few additions whose roundings a product's error could hide behind
SHORT_SUMS = [(18, 1, 96, 170, 48, 5), (9, 8, 94, 77, 16, 2), (6, 7, 60, 70, 33, 2), (4, 3, 80, 90, 40, 3), (5, 4, 50, 61, 20, 3), (3, 10, 50, 64, 64, 2)]


@pytest.mark.parametrize("shape", SHORT_SUMS, ids=ids)
def test_short_sums_are_no_further_off_than_on_the_fp32_kernel(shape):
    N, C, H, W, K, F = shape
    T = C * F * F
    x, f = wl.random_case(9420 + T, *shape)
    acc, mag, _ = oracle.general(x, f)
    got, fp32 = (call(x, f, v) for v in (dconv.VARIANT_FEW_CHANNELS, dconv.VARIANT_TILED))
    assert_within_bound(got, acc, mag, f"few taps {shape}")
    err = np.linalg.norm(got - acc), np.linalg.norm(fp32 - acc)
    print(f"  {T} taps: {err[0] / np.linalg.norm(acc):.3g} against {err[1] / np.linalg.norm(acc):.3g}")
    assert err[0] <= err[1], err
    # one value a channel and a weight a filter: what a product leaves out is the same in all terms of a sum
    x[:] = np.random.default_rng(T).uniform(0.5, 2, (1, C, 1, 1))
    f[:] = np.random.default_rng(T + 1).uniform(0.5, 2, (K, 1, 1, 1))
    acc, mag, _ = oracle.general(x, f)
    # (2^-24 a product; the large products' sum is rounded every eight of them, the small ones' sum counts for 2^-8 of it,
    # and both are added)
    assert np.all(np.abs(call(x, f, dconv.VARIANT_FEW_CHANNELS) - acc) <= 2.0 ** -24 * (1 + 1.2 * -(-T // 8) + 1) * mag)


# layers that the rule sends there: filters that stay on the chip, filters that go through the workspace
CHOSEN = [(1, 1, 720, 1280, 40, 9), (1, 1, 409, 724, 130, 9), (20, 3, 150, 148, 64, 5), (12, 3, 150, 148, 64, 11)]
THROUGH_THE_WORKSPACE = CHOSEN[3]


@pytest.mark.parametrize("shape", CHOSEN, ids=ids)
def test_where_the_library_picks_it(shape):
    assert dconv.kernel_choice(False, *shape) == FEW_CHANNELS
    x, f = map(dev, wl.random_case(9440, *shape))
    want = dconv.dconv_general(x, f, variant=FEW_CHANNELS)
    assert torch.equal(dconv.dconv_general(x, f), want) and torch.equal(dconv.dconv_general(x, f, noalloc=True), want)
    if shape[:2] == (1, 1):
        assert dconv.kernel_choice(True, *shape) == FEW_CHANNELS
        assert torch.equal(dconv.dconv_single_channel(x[0, 0], f[:, 0].contiguous()), want[0])


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("shape", CHOSEN, ids=ids)
def test_captured_calls(shape, noalloc):
    """A graph replays the eager call's bits where the filters stay on the chip or the scratch memory is the static
    array; else those of the kernel that runs in its place."""
    x, f = map(dev, wl.random_case(9450, *shape))
    out = torch.empty_like(dconv.dconv_general(x, f))
    replaced = shape == THROUGH_THE_WORKSPACE and not noalloc
    s, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        eager = dconv.dconv_general(x, f, noalloc=noalloc)
    s.synchronize()
    want = dconv.dconv_general(x, f, variant=dconv.VARIANT_TILED) if replaced else eager
    print(f"capturing {shape} noalloc={noalloc}", flush=True)
    with torch.cuda.graph(g, stream=s):
        dconv.dconv_general(x, f, out=out, noalloc=noalloc)
    for rep in range(3):
        out.fill_(float("nan"))
        other = dconv.dconv_general(x, f)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want), f"replay {rep}"
        assert replaced or torch.equal(other, want)


def test_two_threads_on_one_stream_through_the_workspace():
    """Both kernels of a call run before another thread's call on the stream overwrites the split filters."""
    cases = [tuple(map(dev, wl.random_case(9460 + i, *shape))) for i, shape in enumerate([THROUGH_THE_WORKSPACE, (9, 3, 120, 130, 48, 11)])]
    want = [dconv.dconv_general(x, f, variant=FEW_CHANNELS) for x, f in cases]
    outs = [[torch.empty_like(w) for _ in range(8)] for w in want]
    s = torch.cuda.Stream()
    torch.cuda.synchronize()

    def work(i):
        with torch.cuda.stream(s):
            for o in outs[i]:
                dconv.dconv_general(*cases[i], out=o, variant=FEW_CHANNELS)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    s.synchronize()
    assert all(torch.equal(o, want[i]) for i in range(2) for o in outs[i])
