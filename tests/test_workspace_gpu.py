"""The workspace of dconv_general over the calls that share it: run once and then captured, captured while the
allocation is let through, used from several graphs, streams and threads.
"""
import ctypes
import threading
import time

import numpy as np
import pytest
import torch

import oracle
import workloads as wl
import paper_1705_10591_amd as dconv
from helpers import assert_within_bound

pytestmark = pytest.mark.gpu

SHARED = dconv.VARIANT_TILED_CFG0 + 2 * 3          # + tile shape: tiles cut over channels
# runs on the split-operand kernel, whole tiles (no counters); on the fp32 kernel its 680 tiles are shared
DEEP = (32, 256, 28, 28, 512, 3)
# on the tiled kernel: parts added by a second kernel, partial sums, no counters; by itself a short launch
ONE_IMAGE = (1, 256, 14, 14, 256, 3)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def make(seed, shape):
    N, C, H, W, K, F = shape
    x, f = wl.random_case(seed, *shape, "u01", "he")
    return x, f, dev(x), dev(f), torch.empty(N, K, H - F + 1, W - F + 1, device="cuda")


def fresh_stream():
    """A stream on which the library holds no workspace."""
    s = torch.cuda.Stream()
    dconv.release_workspace()
    return s


def test_a_layer_run_once_and_then_captured_on_another_kernel():
    """Captured calls stay on the fp32 kernel, which shares this layer's tiles: the block that the call before
    it was given has the counters for that."""
    x, f, xd, fd, out = make(8500, DEEP)
    want = dconv.dconv_general(xd, fd, variant=SHARED + dconv.tile_choice(False, *DEEP))
    s = fresh_stream()
    with torch.cuda.stream(s):
        eager = dconv.dconv_general(xd, fd)
    s.synchronize()
    assert not torch.equal(eager, want), "the split-operand kernel is expected to run here"
    g = torch.cuda.CUDAGraph()
    print(f"capturing {DEEP}", flush=True)
    with torch.cuda.graph(g, stream=s):
        dconv.dconv_general(xd, fd, out=out)
    for rep in range(3):
        out.fill_(float("nan"))
        with torch.cuda.stream(s):
            again = dconv.dconv_general(xd, fd)
        s.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want) and torch.equal(again, eager), f"replay {rep}"
    for n in (0, DEEP[0] - 1):
        acc, mag, _ = oracle.general(np.ascontiguousarray(x[n:n + 1]), f)
        assert_within_bound(out[n:n + 1].cpu().numpy(), acc, mag, f"captured, image {n}")
        assert_within_bound(eager[n:n + 1].cpu().numpy(), acc, mag, f"eager, image {n}")


@pytest.mark.parametrize("kernel", [dconv.VARIANT_TILED, dconv.VARIANT_AUTO])
def test_a_call_without_counters_prepares_the_stream_for_one_with_counters(kernel):
    """The first call that needs the workspace brings all of it, and so does a short launch in place of tiles that
    would be shared."""
    assert dconv.kernel_choice(False, *ONE_IMAGE) == dconv.VARIANT_SHORT
    first, second = make(8501, ONE_IMAGE), make(8502, (3, 16, 28, 28, 130, 3))
    want = dconv.dconv_general(second[2], second[3], variant=SHARED + 1)
    s = fresh_stream()
    with torch.cuda.stream(s):
        dconv.dconv_general(first[2], first[3], variant=kernel)
    s.synchronize()
    g = torch.cuda.CUDAGraph()
    print("capturing shared tiles after parts without counters", flush=True)
    with torch.cuda.graph(g, stream=s):
        dconv.dconv_general(second[2], second[3], out=second[4], variant=SHARED + 1)
    for rep in range(3):
        second[4].fill_(float("nan"))
        dconv.dconv_general(first[2], first[3], variant=kernel)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(second[4], want), f"replay {rep}"


# the kernels that need no workspace where the general kernel would share its tiles: short launches, the taps of few
# filters
WITHOUT = [(ONE_IMAGE, dconv.VARIANT_SHORT), ((16, 200, 40, 64, 3, 3), dconv.VARIANT_FEW_TAPS)]


@pytest.mark.parametrize("shape,kernel", WITHOUT, ids=["short", "few_taps"])
def test_what_a_stream_was_given_is_asked_for_again_after_a_release(shape, kernel):
    """Such a call prepares the stream for a captured one that needs the workspace, every time that it has none: the
    second call on a stream asks for nothing, the first one after a release does."""
    assert dconv.kernel_choice(False, *shape) == kernel
    first, second = make(8520, shape), make(8521, (3, 16, 28, 28, 130, 3))
    want = dconv.dconv_general(second[2], second[3], variant=SHARED + 1)
    s = torch.cuda.Stream()
    for rep in range(2):
        torch.cuda.synchronize()
        dconv.release_workspace()
        with torch.cuda.stream(s):
            eager = [dconv.dconv_general(first[2], first[3]) for _ in range(2)]
        s.synchronize()
        assert torch.equal(*eager)
        g = torch.cuda.CUDAGraph()
        print(f"capturing after {shape}, time {rep}", flush=True)
        with torch.cuda.graph(g, stream=s):
            dconv.dconv_general(second[2], second[3], out=second[4], variant=SHARED + 1)
        for _ in range(2):
            second[4].fill_(float("nan"))
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(second[4], want), f"time {rep}"
        del g


def test_a_capture_that_lets_the_allocation_through_leaves_cleared_counters():
    """In relaxed mode a first call may allocate while it is captured: calls before the first replay find cleared
    counters, and replays do not clear them again."""
    x, f, xd, fd, out = make(8503, (3, 16, 28, 28, 130, 3))
    want = dconv.dconv_general(xd, fd, variant=SHARED + 1)
    torch.cuda.synchronize()
    s = fresh_stream()
    g = torch.cuda.CUDAGraph()
    print("capturing a first call in relaxed mode", flush=True)
    with torch.cuda.graph(g, stream=s, capture_error_mode="relaxed"):
        dconv.dconv_general(xd, fd, out=out, variant=SHARED + 1)
    for rep in range(3):
        with torch.cuda.stream(s):
            eager = dconv.dconv_general(xd, fd, variant=SHARED + 1)
        s.synchronize()
        assert torch.equal(eager, want), f"eager call {rep}"
        out.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want), f"replay {rep}"


def test_a_graph_runs_on_one_stream_beside_calls_on_the_stream_it_was_captured_on():
    """Captured launches have a block of their own: the partial sums of a replay and the split filters of calls
    made meanwhile on the capture stream do not meet."""
    a, b = make(8504, (3, 64, 40, 44, 130, 3)), make(8505, (14, 48, 66, 66, 64, 4))
    want_a = dconv.dconv_general(a[2], a[3], variant=SHARED + 1)
    want_b = dconv.dconv_general(b[2], b[3])
    outs = [torch.empty_like(a[4]) for _ in range(10)]
    s, other = fresh_stream(), torch.cuda.Stream()
    with torch.cuda.stream(s):
        dconv.dconv_general(a[2], a[3], variant=SHARED + 1)
    s.synchronize()
    g = torch.cuda.CUDAGraph()
    print("capturing ten launches", flush=True)
    with torch.cuda.graph(g, stream=s):
        for o in outs:
            dconv.dconv_general(a[2], a[3], out=o, variant=SHARED + 1)
    results = [torch.empty_like(b[4]) for _ in range(30)]
    torch.cuda.synchronize()
    for rep in range(3):
        for t in outs + results:
            t.fill_(float("nan"))
        torch.cuda.synchronize()
        for i in range(5):
            with torch.cuda.stream(other):
                g.replay()
            with torch.cuda.stream(s):
                for o in results[6 * i:6 * i + 6]:
                    dconv.dconv_general(b[2], b[3], out=o)
        torch.cuda.synchronize()
        assert all(torch.equal(o, want_a) for o in outs), f"replays, {rep}"
        assert all(torch.equal(o, want_b) for o in results), f"calls, {rep}"


def test_the_per_thread_stream_has_a_workspace_for_every_thread():
    """hipStreamPerThread is one handle and another stream in each thread: the split filters and the partial
    sums of two threads' calls do not meet.  Threads that follow take over what ended threads left, which
    may still be at work."""
    lib, per_thread, vp = dconv.load_library(), ctypes.c_void_p(2), ctypes.c_void_p
    cases = [(shape, make(8510 + i, shape)) for i, shape in enumerate(
        ((14, 48, 66, 66, 64, 4), (6, 48, 40, 44, 100, 6), (1, 256, 14, 14, 256, 3), (2, 64, 30, 30, 64, 3)))]
    wants = [dconv.dconv_general(c[2], c[3]) for _, c in cases]
    outs = [[torch.empty_like(c[4]) for _ in range(12)] for _, c in cases]
    torch.cuda.synchronize()
    dconv.release_workspace()
    errors = []

    def work(i, go, hold):
        (N, C, H, W, K, F), (_, _, xd, fd, _) = cases[i]
        go.wait()
        for o in outs[i]:
            rc = lib.dconv_general(vp(xd.data_ptr()), N, C, H, W, vp(fd.data_ptr()), K, F, vp(o.data_ptr()), per_thread)
            if rc != dconv.STATUS_OK:
                errors.append((i, rc))
        hold.wait()

    def run(together):
        for t in sum(outs, []):
            t.fill_(float("nan"))
        torch.cuda.synchronize()
        go, hold = threading.Barrier(len(cases) if together else 1), threading.Event()
        threads = [threading.Thread(target=work, args=(i, go, hold)) for i in range(len(cases))]
        if not together:
            hold.set()
        for t in threads:
            t.start()
            if not together:
                t.join()
        if together:
            torch.cuda.synchronize()
        hold.set()
        for t in threads:
            t.join()
        # (a device synchronisation does not wait for the streams of threads that have ended)
        deadline = time.time() + 20
        while any(bool(torch.isnan(o).any()) for o in sum(outs, [])) and time.time() < deadline:
            time.sleep(0.01)
        assert not errors, errors
        for i, want in enumerate(wants):
            assert all(torch.equal(o, want) for o in outs[i]), f"{cases[i][0]}, together={together}"
        return torch.cuda.mem_get_info()[0]

    left = []
    for rep in range(3):
        print(f"four threads on the per-thread stream, one after the other and together, {rep}", flush=True)
        run(False)
        left.append(run(True))
    # 24 threads, at most four at a time: not 24 blocks (a thread may begin while the one before it, joined, ends)
    assert left[0] - left[2] <= 4 * (65 << 20), "the threads' blocks are used again"


def test_a_first_call_does_not_disturb_a_capture_on_another_stream():
    """The first call of a large layer on a stream allocates its workspace; a capture going on elsewhere, in the
    default mode, stays valid."""
    shape = (1, 64, 224, 224, 64, 3)            # (whole tiles on the fp32 kernel: no workspace there)
    x, f, xd, fd, out = make(8520, shape)
    x1, f1, xd1, fd1, out1 = make(8521, (2, 8, 30, 30, 70, 3))
    want, want1 = dconv.dconv_general(xd, fd), dconv.dconv_general(xd1, fd1)
    N, C, H, W, K, F = shape
    s, vp = fresh_stream(), ctypes.c_void_p
    g, capturing = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    print("a first call on a stream beside a capture", flush=True)
    with torch.cuda.graph(g, stream=capturing):
        dconv.dconv_general(xd1, fd1, out=out1)
        rc = dconv.load_library().dconv_general(vp(xd.data_ptr()), N, C, H, W, vp(fd.data_ptr()), K, F, vp(out.data_ptr()),
                                                vp(s.cuda_stream))
        dconv.dconv_general(xd1, fd1, out=out1)
    assert rc == dconv.STATUS_OK
    s.synchronize()
    assert torch.equal(out, want)
    for rep in range(3):
        out1.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out1, want1), f"replay {rep}"
