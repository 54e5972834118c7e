"""The split-operand kernel of the general case: fp32 layers on the bf16 matrix cores, each value as
three bf16 parts.  The library picks it by size (3x3 and neighbouring filters, enough work), so the
shapes here are ones it is picked for: a call that ran on it differs in its last bits from the
fp32 matrix-core kernel with the library's own schedule (VARIANT_TILED) and is closer to the exact sums.
"""
import ctypes
import threading

import numpy as np
import pytest
import torch

import oracle
import workloads as wl
import paper_1705_10591_amd as dconv
from helpers import assert_within_bound

pytestmark = pytest.mark.gpu

# (N, C, H, W, K, F): every compiled filter side; channels off multiples of sixteen (zero channels in
# the last chunk), filters off multiples of 64, column strips, pixel tiles that end anywhere in a
# row, whole tiles and tiles shared between workgroups
SHAPES = [(11, 154, 63, 63, 39, 2), (4, 96, 55, 55, 179, 3), (20, 61, 65, 65, 64, 3), (2, 100, 60, 300, 120, 3),
          (1, 64, 224, 224, 64, 3), (14, 48, 66, 66, 64, 4), (5, 40, 75, 67, 100, 5), (6, 48, 40, 44, 100, 6),
          (3, 40, 60, 62, 120, 7), (8, 97, 25, 25, 250, 7)]
ids = lambda s: "x".join(map(str, s))


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def call(x, f, variant=dconv.VARIANT_AUTO, noalloc=False):
    print(f"general {tuple(x.shape)} K,F={f.shape[0]},{f.shape[-1]} variant={variant:#x}", flush=True)
    out = dconv.dconv_general(dev(x), dev(f), variant=variant, noalloc=noalloc)
    torch.cuda.synchronize()
    return out.cpu().numpy()


# the fp32 kernel with the shape's own tile and schedule
FP32 = dconv.VARIANT_TILED


@pytest.mark.parametrize("shape", SHAPES, ids=ids)
def test_within_the_bound_and_closer_than_the_fp32_kernel(shape):
    N, C, H, W, K, F = shape
    x, f = wl.random_case(8000 + C + F, N, C, H, W, K, F, "u01", "he")
    acc, mag, _ = oracle.general(x, f)
    got, fp32 = call(x, f), call(x, f, FP32)
    assert not np.array_equal(got, fp32), "the split-operand kernel is expected to run here"
    assert_within_bound(got, acc, mag, f"split {shape}")
    err = np.linalg.norm(got - acc), np.linalg.norm(fp32 - acc)
    assert err[0] <= err[1], err
    # the same bits every time and through both entry points; a forced configuration is the fp32 kernel's
    assert np.array_equal(call(x, f), got) and np.array_equal(call(x, f, noalloc=True), got)
    assert np.array_equal(call(x, f, dconv.VARIANT_TILED_CFG0 + dconv.tile_choice(False, *shape)), fp32)


@pytest.mark.parametrize("shape", SHAPES, ids=ids)
def test_integer_inputs_exact_between_guard_bands(shape):
    N, C, H, W, K, F = shape
    x, f = wl.integer_case(8100 + C + F, N, C, H, W, K, F)
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


@pytest.mark.parametrize("shape", [(4, 96, 55, 55, 179, 3), (14, 48, 66, 66, 64, 4), (3, 40, 60, 62, 120, 7)], ids=ids)
def test_values_the_parts_cannot_carry(shape):
    """Infinities, NaN, values next to the largest float, subnormal values and products of tiny and huge
    ones: the outputs they reach are what fp32 gives, the others are untouched."""
    N, C, H, W, K, F = shape
    x, f = wl.random_case(8200 + F, N, C, H, W, K, F)
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
    # (the reference result of a subnormal product may be off by half the smallest float a term)
    for sx, sf in ((2.0**-120, 1.0), (2.0**-128, 2.0**20), (1.0, 2.0**-118), (2.0**-115, 2.0**60), (2.0**70, 2.0**-130)):
        xs, fs = (x * np.float32(sx)).astype(np.float32), (f * np.float32(sf)).astype(np.float32)
        acc, mag, _ = oracle.general(xs, fs)
        got = call(xs, fs)
        assert np.all(np.abs(got - acc) <= 1e-5 * mag + C * F * F * 2.0**-150), (sx, sf)
    # half of the images far below the other half
    xs = x.copy()
    xs[::2] *= np.float32(2.0**-122)
    acc, mag, _ = oracle.general(xs, f)
    got = call(xs, f)
    assert np.all(np.abs(got - acc) <= 1e-5 * mag + C * F * F * 2.0**-150)


@pytest.mark.parametrize("shape", [(14, 48, 66, 66, 64, 4), (3, 40, 60, 62, 120, 7)], ids=ids)
def test_a_sum_of_one_term_is_within_one_unit_in_the_last_place(shape):
    """Filters of one weight: an output is one product.  Its three smallest products of parts, 2^-24 of it at
    most, are left out and the rest is rounded: at most one unit in the last place.  Weights of eight bits
    and VARIANT_TILED: the product rounded once."""
    N, C, H, W, K, F = shape
    rng = np.random.default_rng(8600 + F)
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    f, at = np.zeros((K, C, F, F), np.float32), []
    for k in range(K):
        at.append((rng.integers(C), rng.integers(F), rng.integers(F)))
        f[(k, *at[-1])] = rng.standard_normal()
    want = np.stack([x[:, c, i:i + H - F + 1, j:j + W - F + 1].astype(np.float64) * f[k, c, i, j] for k, (c, i, j) in enumerate(at)], axis=1)
    got = call(x, f)
    ulp = np.spacing(np.abs(want).astype(np.float32)).astype(np.float64)
    off = np.abs(got - want) / ulp
    print(f"split {shape}: {off.max():.3f} units in the last place, rms {np.sqrt((off ** 2).mean()):.3f}", flush=True)
    assert not np.array_equal(got, want.astype(np.float32)) and off.max() <= 1.0
    assert np.array_equal(call(x, f, FP32), want.astype(np.float32))
    short = (f.view(np.uint32) & np.uint32(0xFFFF0000)).view(np.float32)      # eight bits: h' alone
    want = np.stack([x[:, c, i:i + H - F + 1, j:j + W - F + 1] * short[k, c, i, j] for k, (c, i, j) in enumerate(at)], axis=1)
    assert np.abs(call(x, short) - want.astype(np.float64)).max() <= (0.502 * np.spacing(np.abs(want))).max()


@pytest.mark.parametrize("shape", [(4, 96, 55, 55, 179, 3), (14, 48, 66, 66, 64, 4)], ids=ids)
def test_products_near_and_below_the_smallest_normal_value(shape):
    """Operands whose parts are all there, products of parts that are subnormal: nothing is formed again, the
    matrix cores keep subnormal products and sums."""
    N, C, H, W, K, F = shape
    x, f = wl.random_case(8700 + F, N, C, H, W, K, F, "u01", "he")
    for sx, sf in ((-56, -56), (-62, -60), (-70, -50), (-75, -66), (-60, -72)):
        xs, fs = np.ldexp(x, sx).astype(np.float32), np.ldexp(f, sf).astype(np.float32)
        assert np.abs(xs[xs != 0]).min() > 2.0 ** -103 and np.abs(fs[fs != 0]).min() > 2.0 ** -103
        acc, mag, _ = oracle.general(xs, fs)
        got = call(xs, fs)
        assert np.all(np.abs(got - acc) <= 1e-5 * mag + C * F * F * 2.0 ** -150), (sx, sf)


def test_values_the_parts_cannot_carry_among_many_tiles():
    """Over a hundred tiles a workgroup: the tiles to be formed again are found by their outputs.  Against the
    fp32 kernel, by the bound that its sums of magnitudes give."""
    shape = (32, 32, 256, 256, 256, 3)
    N, C, H, W, K, F = shape
    g = torch.Generator(device="cuda").manual_seed(82)
    x = torch.rand((N, C, H, W), generator=g, device="cuda")
    f = torch.randn((K, C, F, F), generator=g, device="cuda") * 0.1
    x[1::2] *= 2.0 ** -112
    mag = dconv.dconv_general(x, f.abs(), variant=FP32)
    for n, c, y, xx in ((0, 0, 0, 0), (6, 31, 255, 255), (6, 3, 100, 31), (31, 17, 254, 1)):
        x[n, c, y, xx] = float("nan")
    x[13, 2, 40, 40] = float("inf")
    print(f"general {shape}", flush=True)
    got, want = dconv.dconv_general(x, f), dconv.dconv_general(x, f, variant=FP32)
    torch.cuda.synchronize()
    fine = torch.isfinite(want)
    assert 0 < int((~fine).sum()) < 10 * 10 * K
    assert torch.equal(torch.isnan(got), torch.isnan(want)) and torch.equal(torch.isinf(got), torch.isinf(want))
    assert not torch.equal(got[0, :, 8:], want[0, :, 8:]), "the split-operand kernel is expected to run here"
    assert bool(((got - want).abs()[fine] <= 2e-5 * mag[fine]).all())


def test_time_does_not_depend_on_the_data_without_bound():
    """One pixel that is not a number: its outputs are formed again, at a small multiple of the call's time
    (2.1 times measured; a lane for each output, one after the other, took 20)."""
    w = wl.G3
    x, f = map(dev, wl.make_inputs(w))
    out = torch.empty(w.out_shape(), device="cuda")

    def us():
        dconv.dconv_general(x, f, out=out)
        best = float("inf")
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            dconv.dconv_general(x, f, out=out)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 1e3)
        return best

    clean = us()
    x[w.N - 1, w.C // 2, w.H // 2, w.W // 2] = float("nan")
    marked = us()
    print(f"{clean:.1f} us, with one NaN {marked:.1f} us", flush=True)
    assert int(torch.isnan(out).sum()) == w.K * w.F * w.F
    assert marked < 6 * clean


def test_two_threads_on_one_stream():
    """The filters are split into the stream's workspace by a kernel of its own: two threads that call
    on one stream must not come between each other's two kernels."""
    lib, stream = dconv.load_library(), torch.cuda.Stream()
    vp, cases = ctypes.c_void_p, []
    for shape in ((14, 48, 66, 66, 64, 4), (6, 48, 40, 44, 100, 6)):
        N, C, H, W, K, F = shape
        x, f = wl.random_case(8300 + F, *shape)
        xd, fd = dev(x), dev(f)
        cases.append((shape, xd, fd, dconv.dconv_general(xd, fd), [torch.empty(N, K, H - F + 1, W - F + 1, device="cuda")
                                                                  for _ in range(20)]))
    torch.cuda.synchronize()

    def work(case):
        (N, C, H, W, K, F), xd, fd, _, outs = case
        for o in outs:
            assert lib.dconv_general(vp(xd.data_ptr()), N, C, H, W, vp(fd.data_ptr()), K, F, vp(o.data_ptr()),
                                     vp(stream.cuda_stream)) == dconv.STATUS_OK

    threads = [threading.Thread(target=work, args=(c,)) for c in cases]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    stream.synchronize()
    for _, _, _, want, outs in cases:
        assert all(torch.equal(o, want) for o in outs)


def test_a_first_call_on_a_stream_can_be_captured():
    """A capture may not allocate: such a call runs on the fp32 kernel, as it did without a workspace."""
    shape = (1, 64, 224, 224, 64, 3)            # (whole tiles on the fp32 kernel: no workspace there)
    N, C, H, W, K, F = shape
    x, f = wl.random_case(8400, *shape)
    acc, mag, _ = oracle.general(x, f)
    xd, fd = dev(x), dev(f)
    out = torch.empty(acc.shape, device="cuda")
    warm = dconv.dconv_general(xd, fd, variant=FP32)      # (loads the kernel; no workspace)
    torch.cuda.synchronize()
    g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    print("capturing a first call", flush=True)
    with torch.cuda.graph(g, stream=s):
        dconv.dconv_general(xd, fd, out=out)
    for rep in range(3):
        out.fill_(float("nan"))
        eager = dconv.dconv_general(xd, fd)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, warm), f"replay {rep}"
        assert_within_bound(eager.cpu().numpy(), acc, mag, "eager call between replays")
