"""Performance cases of the library: what a user of dconv has it do, through the public calls.

A case is a dict: `entry` ("single", "general", "half", "i8"), the sizes of the C ABI (batch N,
channels C, image H x W, K filters of F x F), the distributions of its inputs and the options of
the call.  Sizes are those of the repository's own workloads (workloads.py) or generic ones.
"""
from __future__ import annotations

import math

import torch

import paper_1705_10591_amd as dconv

_HALF = {"f16": torch.float16, "bf16": torch.bfloat16}


def _case(name, entry, N, C, H, W, K, F, dtype="f32", dist="u01", blocked=False, noalloc=False):
    return {"name": name, "entry": entry, "N": N, "C": C, "H": H, "W": W, "K": K, "F": F,
            "dtype": dtype, "dist": dist, "blocked": blocked, "noalloc": noalloc}


def listed():
    return [
        # one small image, a small bank of 3x3 filters: a call of a few microseconds, where the
        # launch and the chain of latencies are the time (workload S1)
        _case("single_256_k16_f3", "single", 1, 1, 256, 256, 16, 3, dist="u11"),
        # the headline workload: one large image, 64 5x5 filters, bound by its 4.3 GB of output (S2)
        _case("single_4096_k64_f5", "single", 1, 1, 4096, 4096, 64, 5, dist="u11"),
        # a bank of 40 oriented filters (five scales, eight directions) on a video frame whose
        # sides are not round numbers
        _case("single_1081x1917_k40_f9", "single", 1, 1, 1081, 1917, 40, 9, dist="u11"),
        # first layer with large filters on a batch of RGB images (G1)
        _case("general_rgb_224_k64_f11", "general", 64, 3, 224, 224, 64, 11, dist="u11"),
        # middle layer of a network, a batch of 32 (G2)
        _case("general_c64_56_k64_f3", "general", 32, 64, 56, 56, 64, 3),
        # deep layer of a network, a batch of 32 (G3)
        _case("general_c256_28_k512_f3", "general", 32, 256, 28, 28, 512, 3),
        # a deep layer for ONE image, called by a serving loop that may not allocate
        _case("general_one_image_c256_14_f3", "general", 1, 256, 14, 14, 256, 3, noalloc=True),
        # last layer of an image-to-image network: features to RGB
        _case("general_to_rgb_c64_224_k3_f3", "general", 8, 64, 224, 224, 3, 3),
        # nothing is a multiple of a tile: batch, channels, map and filter count off the round sizes
        _case("general_ragged_c40_75x67_k100_f5", "general", 5, 40, 75, 67, 100, 5),
        # the deep layer with 16-bit inputs, channels last
        _case("bf16_c256_28_k512_f3", "half", 32, 256, 28, 28, 512, 3, dtype="bf16"),
        # a 1x1 (bottleneck) layer with 16-bit inputs, channels last
        _case("f16_c512_28_k128_f1", "half", 32, 512, 28, 28, 128, 1, dtype="f16"),
        # a quantised layer, channel-blocked layout
        _case("i8_blocked_c128_56_k128_f3", "i8", 32, 128, 56, 56, 128, 3, dtype="i8", blocked=True),
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case: an image and a filter bank; a layer in fp32 (first layers on few channels, few
    filters, deep layers on small maps, one image or a batch); a layer in 16 or 8 bits."""
    while True:
        family = rng.choice(["single", "first", "layer", "layer", "layer", "few", "half", "half", "i8"])
        side = 3 if rng.random() < 0.4 else rng.choice([1, 2, 3, 4, 5, 7, 9, 11])
        if family == "single":
            H, W = _log(rng, 64, 4096), _log(rng, 64, 4096)
            c = _case("", "single", 1, 1, H, W, _log(rng, 1, 256), side, dist="u11")
        elif family == "first":
            C = rng.choice([1, 2, 3, 3, 3, 4])
            c = _case("", "general", _log(rng, 1, 64), C, _log(rng, 28, 512), _log(rng, 28, 512),
                      rng.choice([16, 32, 48, 64, 64, 96, 128]), side, dist="u11")
        elif family in ("layer", "few"):
            C = _log(rng, 5, 512)
            if rng.random() < 0.5:
                C = max(16, C // 16 * 16)
            few = family == "few"
            K = rng.randint(1, 12) if few else _log(rng, 16, 512)
            if not few and rng.random() < 0.5:
                K = max(16, K // 16 * 16)
            H = _log(rng, 28 if few else 7, 256 if few else 128)
            W = max(7, min(512, int(round(H * rng.choice([1.0, 1.0, rng.uniform(0.5, 2.0)])))))
            c = _case("", "general", _log(rng, 1, 64), C, H, W, K, min(side, 7 if few else 11),
                      noalloc=rng.random() < 0.2)
        else:
            step = 16 if family == "half" else 32
            H = _log(rng, 7, 128)
            W = max(7, int(round(H * rng.choice([1.0, 1.0, rng.uniform(0.5, 2.0)]))))
            dtype = rng.choice(["f16", "bf16"]) if family == "half" else "i8"
            c = _case("", family, _log(rng, 1, 64), step * _log(rng, 1, 512 // step), H, W,
                      _log(rng, 16, 512), min(side, 7), dtype=dtype, blocked=rng.random() < 0.4)
        if c["F"] > min(c["H"], c["W"]):
            continue
        w = work(c)
        # no dearer than the largest listed cases: 136 GFLOP in fp32, 4.4 GB
        if w["flops"] <= 1.3e11 and w["bytes"] <= 2.2e9:
            del c["name"]
            return c


def _inputs(case, seed):
    """Image(s) and filters on the GPU in the plain layout, as the values the call is to see: fp32 in
    [-1, 1) (signals) or activations in [0, 1) with He-distributed filters; 8-bit integers."""
    N, C, H, W, K, F = (case[k] for k in "NCHWKF")
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    if case["dtype"] == "i8":
        x = torch.randint(0, 128, (N, C, H, W), generator=g, device="cuda", dtype=torch.int8)
        f = torch.randint(-127, 128, (K, C, F, F), generator=g, device="cuda", dtype=torch.int8)
        return x, f
    x = torch.rand((N, C, H, W), generator=g, device="cuda")
    if case["dist"] == "u11":
        x = x * 2.0 - 1.0
        f = torch.rand((K, C, F, F), generator=g, device="cuda") * 2.0 - 1.0
    else:
        f = torch.randn((K, C, F, F), generator=g, device="cuda") * math.sqrt(2.0 / (C * F * F))
    if case["dtype"] in _HALF:
        x, f = x.to(_HALF[case["dtype"]]), f.to(_HALF[case["dtype"]])
    return x, f


def _lay_out(t, case):
    """[A, C, h, w] -> channels last [A, h, w, C], or channel-blocked [A, C/cb, h, w, cb]."""
    if not case["blocked"]:
        return t.permute(0, 2, 3, 1).contiguous()
    cb = 32 // t.element_size()
    A, C, h, w = t.shape
    return t.view(A, C // cb, cb, h, w).permute(0, 1, 3, 4, 2).contiguous()


def prepare(case, seed):
    x, f = _inputs(case, seed)
    if case["entry"] == "single":
        x, f = x[0, 0].contiguous(), f[:, 0].contiguous()
    elif case["entry"] in ("half", "i8"):
        x, f = _lay_out(x, case), _lay_out(f, case)
    state = {"case": case, "x": x, "f": f, "out": None}
    if case["noalloc"]:
        shape = (case["N"], case["K"], case["H"] - case["F"] + 1, case["W"] - case["F"] + 1)
        state["out"] = torch.empty(shape, dtype=torch.float32, device="cuda")
    return state


def run(state):
    case, x, f = state["case"], state["x"], state["f"]
    if case["entry"] == "single":
        return dconv.dconv_single_channel(x, f)
    if case["entry"] == "general":
        return dconv.dconv_general(x, f, out=state["out"], noalloc=case["noalloc"])
    if case["entry"] == "half":
        return dconv.dconv_general_half(x, f, blocked=case["blocked"])
    return dconv.dconv_general_i8(x, f, blocked=case["blocked"])


def work(case):
    """Each input read once, each output written once; a multiply and an add per tap."""
    N, C, H, W, K, F = (case[k] for k in "NCHWKF")
    out = N * K * (H - F + 1) * (W - F + 1)
    size = {"f32": 4, "f16": 2, "bf16": 2, "i8": 1}[case["dtype"]]
    return {"bytes": size * (N * C * H * W + K * C * F * F) + 4 * out, "flops": 2 * out * C * F * F}


def tolerance(case):
    # Outputs are 32-bit sums of exact (8- and 16-bit inputs) or 24-bit products, whatever the
    # order of the additions; whole numbers are exact.  Measured against `exact` on the listed
    # cases and twelve drawn ones: relative error up to 7.5e-7, largest error up to 6.8e-6.
    if case["dtype"] == "i8":
        return "exact"
    return {"rel": 3e-6, "max": 3e-5}


def exact(case, seed):
    x, f = _inputs(case, seed)
    N, C, H, W, K, F = (case[k] for k in "NCHWKF")
    Ho, Wo = H - F + 1, W - F + 1
    xt = x.permute(1, 0, 2, 3).to(torch.float64)
    ft = f.to(torch.float64)
    acc = torch.zeros((K, N * Ho * Wo), dtype=torch.float64, device="cuda")
    for i in range(F):
        for j in range(F):
            acc.addmm_(ft[:, :, i, j].contiguous(), xt[:, :, i:i + Ho, j:j + Wo].reshape(C, -1))
    out = acc.view(K, N, Ho, Wo).permute(1, 0, 2, 3)
    if case["dtype"] == "i8":
        return out.round().to(torch.int32).contiguous()
    return out[0].contiguous() if case["entry"] == "single" else out.contiguous()
