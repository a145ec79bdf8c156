"""Stream semantics of the C ABI on the GPU: every entry point enqueues on the stream it is given and returns
without synchronising, multi-launch plans stay ordered on that stream, streams and host threads may share a context,
and a call whose scratch is already sized can be captured into a HIP graph and replayed (results compared with eager
calls and with the oracle).
"""
import ctypes
import threading

import numpy as np
import pytest

from paper_2501_08455_amd import workloads
from test_gpu_backward import launches
from test_gpu_parity import TOL, gpu, level_errors, say  # noqa: F401  (gpu is a fixture)

pytestmark = pytest.mark.gpu


def plans(gpu):
    return {
        "auto": None,
        "two segments (fold + join launches)": gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, prefix_depth=2, chunks=4, segments=2),
        "level-scan (one launch per level)": gpu.make_plan(gpu.SIG_VARIANT_LEVEL_SCAN, chunks=0),
        "HBM streaming": gpu.make_plan(gpu.SIG_VARIANT_HBM_STREAMING, prefix_depth=1),
    }


def test_calls_on_a_side_stream(gpu, oracle):
    import torch
    x = workloads.brownian_paths(40, 400, 5, seed=91)
    want = oracle.signature(x, 4)
    side = torch.cuda.Stream()           # default priority
    ctx = gpu.sig_create()
    try:
        xt = torch.from_numpy(x).cuda()
        torch.cuda.synchronize()
        for label, plan in plans(gpu).items():
            out = torch.full((40, gpu.sig_size(5, 4)), float("nan"), device="cuda")
            torch.cuda.synchronize()
            with torch.cuda.stream(side):
                assert gpu.sig_compute(ctx, xt, 4, 0, out, stream=side, plan=plan) == gpu.SIG_OK
                # a consumer on the same stream sees the finished result without any host synchronisation
                total = out.sum()
            side.synchronize()
            errs = level_errors(out.cpu().numpy(), want, 5, 4)
            say("  side stream, %s: %s" % (label, " ".join("%.2e" % e for e in errs)))
            assert max(errs) <= TOL and bool(torch.isfinite(total))
    finally:
        torch.cuda.synchronize()
        gpu.sig_destroy(ctx)


def test_backward_on_a_side_stream(gpu, oracle):
    import torch
    side = torch.cuda.Stream()
    ctx = gpu.sig_create()
    try:
        # on brackets (one launch; the third cut across workgroups), then the two-launch sliced sweep and the sweep cut into time
        # segments (eight launches)
        for d, depth, B, L in [(5, 4, 9, 60), (10, 4, 3, 20), (8, 4, 2, 300), (10, 5, 3, 20), (7, 5, 2, 300)]:
            x = workloads.brownian_paths(B, L, d, seed=92 + d)
            g = np.random.default_rng(d).normal(size=(B, gpu.sig_size(d, depth))).astype(np.float32)
            want = oracle.signature_backward(x, depth, g)
            xt, gt = torch.from_numpy(x).cuda(), torch.from_numpy(g).cuda()
            out = torch.empty((B, gpu.sig_size(d, depth)), device="cuda")
            gx = torch.full(x.shape, float("nan"), device="cuda")
            torch.cuda.synchronize()
            with torch.cuda.stream(side):
                assert gpu.sig_compute(ctx, xt, depth, 0, out, stream=side) == gpu.SIG_OK
                assert gpu.sig_backward(ctx, xt, depth, 0, out, gt, gx, stream=side) == gpu.SIG_OK
            side.synchronize()
            got = gx.cpu().numpy()
            err = np.linalg.norm(got - want) / np.linalg.norm(want)
            say("  backward on a side stream (%d, %d): %.2e" % (d, depth, err))
            assert err <= TOL
    finally:
        torch.cuda.synchronize()
        gpu.sig_destroy(ctx)


def test_graph_capture_and_replay(gpu, oracle):
    """The calls allocate nothing once the context's scratch is sized, so they can be captured.  Every replay is
    checked against the eager result, with new input values and eager work between the replays."""
    import torch
    B, L, d, depth = 24, 300, 5, 4
    ctx = gpu.sig_create()
    try:
        xs = [workloads.brownian_paths(B, L, d, seed=93 + i) for i in range(3)]
        xt = torch.from_numpy(xs[0]).cuda()
        for label, plan in plans(gpu).items():
            out = torch.zeros((B, gpu.sig_size(d, depth)), device="cuda")
            # eager call first: sizes the scratch (no allocation may happen under capture)
            assert gpu.sig_compute(ctx, xt, depth, 0, out, plan=plan) == gpu.SIG_OK
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                rc = gpu.sig_compute(ctx, xt, depth, 0, out, plan=plan)
            assert rc == gpu.SIG_OK
            for i, x in enumerate(xs):
                xt.copy_(torch.from_numpy(x).cuda())
                out.fill_(float("nan"))
                torch.cuda.synchronize()
                graph.replay()
                torch.cuda.synchronize()
                replayed = out.clone()
                assert gpu.sig_compute(ctx, xt, depth, 0, out, plan=plan) == gpu.SIG_OK
                torch.cuda.synchronize()
                assert torch.equal(replayed, out), (label, i)
                errs = level_errors(replayed.cpu().numpy(), oracle.signature(x, depth), d, depth)
                assert max(errs) <= TOL
            say("  graph replay, %s: three replays equal the eager calls bit for bit" % label)
            xt.copy_(torch.from_numpy(xs[0]).cuda())
    finally:
        torch.cuda.synchronize()
        gpu.sig_destroy(ctx)


@pytest.mark.parametrize("B,L,d,depth,gradient_launches", [(2, 900, 10, 4, 1), (2, 600, 7, 5, 6)])
def test_graph_capture_of_the_paths_cut_in_time(gpu, oracle, B, L, d, depth, gradient_launches):
    """The paths for few long paths — forward segments joined in device memory by several launches, and the gradient cut in
    time, on brackets in one launch and on signatures in six or more — captured together and replayed with new inputs."""
    import torch
    D = gpu.sig_size(d, depth)
    ctx = gpu.sig_create()
    try:
        rc, pl = gpu.sig_plan(ctx, B, L, d, depth, 0)
        assert rc == gpu.SIG_OK and pl.variant == gpu.SIG_VARIANT_ON_CHIP and pl.segments >= 4
        assert gpu.sig_backward_segments(ctx, B, L, d, depth, 0) > 1
        xs = [workloads.brownian_paths(B, L, d, seed=96 + i) for i in range(3)]
        g = np.random.default_rng(5).normal(size=(B, D)).astype(np.float32)
        xt, gt = torch.from_numpy(xs[0]).cuda(), torch.from_numpy(g).cuda()
        out, gx = torch.zeros((B, D), device="cuda"), torch.zeros(xs[0].shape, device="cuda")

        def both():
            assert gpu.sig_compute(ctx, xt, depth, 0, out) == gpu.SIG_OK
            assert gpu.sig_backward(ctx, xt, depth, 0, out, gt, gx) == gpu.SIG_OK

        both()   # sizes the scratch
        assert launches(gpu, lambda: gpu.sig_compute(ctx, xt, depth, 0, out)) >= 4
        n = launches(gpu, lambda: gpu.sig_backward(ctx, xt, depth, 0, out, gt, gx))
        assert n == 1 if gradient_launches == 1 else n >= gradient_launches
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            both()
        for i, x in enumerate(xs):
            xt.copy_(torch.from_numpy(x).cuda())
            out.fill_(float("nan"))
            gx.fill_(float("nan"))
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            r_out, r_gx = out.clone(), gx.clone()
            both()
            torch.cuda.synchronize()
            assert torch.equal(r_out, out) and torch.equal(r_gx, gx), i
            assert max(level_errors(r_out.cpu().numpy(), oracle.signature(x, depth), d, depth)) <= TOL
            want = oracle.signature_backward(x, depth, g)
            assert np.linalg.norm(r_gx.cpu().numpy() - want) / np.linalg.norm(want) <= TOL
        say("  graph replay, paths cut in time: three replays equal the eager calls bit for bit")
    finally:
        torch.cuda.synchronize()
        gpu.sig_destroy(ctx)


def test_pointers_that_are_only_float_aligned(gpu, oracle):
    """The ABI asks for float32 arrays, not for 16-byte alignment: every family, and the gradient, with path, output and
    gradient buffers that start 4 bytes past a 16-byte boundary."""
    import torch

    def shifted(shape, fill=None):
        n = int(np.prod(shape))
        raw = torch.empty(n + 1, dtype=torch.float32, device="cuda")
        view = raw[1:].view(*shape)
        assert view.data_ptr() % 16 == 4
        if fill is not None:
            view.copy_(torch.from_numpy(fill))
        return view

    ctx = gpu.default_ctx()
    cases = [("C1", None), ("C2", None), ("C4", None),
             ("C2", gpu.make_plan(gpu.SIG_VARIANT_LEVEL_SCAN, chunks=0)), ("C4", gpu.make_plan(gpu.SIG_VARIANT_LEVEL_SCAN, chunks=0)),
             ("C4", gpu.make_plan(gpu.SIG_VARIANT_HBM_STREAMING, prefix_depth=1)),
             ("C2", gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, prefix_depth=2, chunks=4, segments=2))]
    for name, plan in cases:
        cfg = workloads.CONFIGS[name]
        x = workloads.make_paths(cfg)[:16]
        B, L, d = x.shape
        D = gpu.sig_size(d, cfg.depth)
        xt = shifted(x.shape, x)
        out = shifted((B, L - 1, D) if cfg.stream else (B, D))
        out.fill_(float("nan"))
        assert gpu.sig_compute(ctx, xt, cfg.depth, int(cfg.stream), out, plan=plan) == gpu.SIG_OK
        torch.cuda.synchronize()
        errs = level_errors(out.cpu().numpy(), oracle.signature(x, cfg.depth, stream=cfg.stream), d, cfg.depth)
        say("  shifted pointers, %s, %s: %s" % (name, "auto" if plan is None else "variant %d" % plan.variant,
                                                " ".join("%.2e" % e for e in errs)))
        assert max(errs) <= TOL
    # gradient: on brackets, also cut across workgroups; register kernel (4, 4) and general sweep (11, 2) in stream mode; on
    # signatures the sliced sweep (10, 5) and the sweep cut into time segments (7, 5), in stream mode (10, 4)
    for d, depth, B, L, stream in [(5, 4, 9, 60, False), (4, 4, 5, 40, True), (10, 4, 3, 20, False), (11, 2, 4, 15, True),
                                   (10, 4, 1, 200, False), (6, 4, 2, 301, False), (10, 5, 2, 20, False), (7, 5, 1, 200, False),
                                   (10, 4, 1, 600, True)]:
        x = workloads.brownian_paths(B, L, d, seed=95 + d)
        D = gpu.sig_size(d, depth)
        rows = (B, L - 1, D) if stream else (B, D)
        g = np.random.default_rng(d).normal(size=rows).astype(np.float32)
        xt, gt, out, gx = shifted(x.shape, x), shifted(rows, g), shifted(rows), shifted(x.shape)
        gx.fill_(float("nan"))
        assert gpu.sig_compute(ctx, xt, depth, int(stream), out) == gpu.SIG_OK
        assert gpu.sig_backward(ctx, xt, depth, int(stream), out, gt, gx) == gpu.SIG_OK
        torch.cuda.synchronize()
        want = oracle.signature_backward(x, depth, g, stream=stream)
        err = np.linalg.norm(gx.cpu().numpy() - want) / np.linalg.norm(want)
        say("  shifted pointers, gradient (%d, %d): %.2e" % (d, depth, err))
        assert err <= TOL


# calls that keep something in context scratch: forward segments joined by a second launch, the level-scan family, the
# gradient cut into time segments, the general gradient, the stretches of rows split across workgroups, the sums of a long path's
# every-prefix gradient at depth 2, the rows that depth 3 of twelve channels leaves for it
SCRATCH = [(128, 2000, 5, 4, 0, False), (48, 200, 12, 3, 1, False), (3, 300, 7, 5, 0, True), (40, 60, 13, 3, 1, True),
           (2, 700, 9, 4, 1, False), (1, 1500, 6, 2, 1, True), (40, 60, 12, 3, 1, True)]


def scratch_call(gpu, ctx, i, seed):
    """Input of call number i and the call itself, as out = call(stream)."""
    import torch
    B, L, d, depth, stream_flag, backward = SCRATCH[i % len(SCRATCH)]
    gen = torch.Generator(device="cuda").manual_seed(seed + i)
    x = (torch.randn(B, L, d, device="cuda", generator=gen) * L ** -0.5).cumsum(1)
    D = gpu.sig_size(d, depth)
    rows = (B, L - 1, D) if stream_flag else (B, D)
    if not backward:
        rc, plan = gpu.sig_plan(ctx, B, L, d, depth, stream_flag)
        plan.row_workgroups = 0   # (rows written straight from registers keep nothing in scratch)
        assert (plan.split_rows > 1) == ((d, depth) == (9, 4))
        rc, _, _, scratch = gpu.sig_plan_footprint(B, L, d, depth, stream_flag, plan)
        assert rc == gpu.SIG_OK and scratch > 0

        def forward(stream):
            out = torch.full(rows, float("nan"), device="cuda")
            if not stream_flag:
                assert gpu.sig_compute(ctx, x, depth, stream_flag, out, stream=stream) == gpu.SIG_OK
            else:
                handle = torch.cuda.ExternalStream(stream) if isinstance(stream, int) else stream
                assert gpu.sig_compute(ctx, x, depth, stream_flag, out, stream=handle, plan=plan) == gpu.SIG_OK
            return out
        return forward
    out, g = torch.empty(rows, device="cuda"), torch.randn(rows, device="cuda", generator=gen)
    assert (gpu.sig_backward_segments(ctx, B, L, d, depth, stream_flag) > 1) == (d != 13)
    assert gpu.sig_compute(ctx, x, depth, stream_flag, out) == gpu.SIG_OK
    torch.cuda.synchronize()

    def gradient(stream):
        gx = torch.full(x.shape, float("nan"), device="cuda")
        assert gpu.sig_backward(ctx, x, depth, stream_flag, out, g, gx, stream=stream) == gpu.SIG_OK
        return gx
    return gradient


def serial(calls):
    import torch
    want = []
    for call in calls:
        want.append(call(torch.cuda.current_stream()))
        torch.cuda.synchronize()
        assert bool(torch.isfinite(want[-1]).all())
    return want


def test_two_streams_share_a_context(gpu):
    """Calls that use the scratch on two streams with nothing to order them but the context: the same bits as one after the
    other.  The streams alternate, then one of them has the context to itself for a while, then they alternate again."""
    import torch
    ctx = gpu.sig_create()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    turns = [0, 1] * 12 + [0] * 70 + [1, 0] * 8
    try:
        for first in range(len(SCRATCH)):
            some = [scratch_call(gpu, ctx, first + i, 200) for i in range(8)]
            calls = [some[i % 8] for i in range(len(turns))]
            torch.cuda.synchronize()
            got = []
            for call, turn in zip(calls, turns):
                with torch.cuda.stream(streams[turn]):
                    got.append(call(streams[turn]))
            torch.cuda.synchronize()
            for i, (a, b) in enumerate(zip(got, serial(calls))):
                assert torch.equal(a, b), (first, i, SCRATCH[(first + i) % len(SCRATCH)])
    finally:
        torch.cuda.synchronize()
        gpu.sig_destroy(ctx)


def test_host_threads_share_a_context(gpu):
    """Four threads, each with a stream of its own, on a context whose scratch has to grow under way."""
    import torch
    calls_ctx, ctx = gpu.sig_create(), gpu.sig_create()
    try:
        n, each = 4, 12
        calls = [[scratch_call(gpu, ctx, t + i, 300 + 50 * t) for i in range(each)] for t in range(n)]
        want = [serial([scratch_call(gpu, calls_ctx, t + i, 300 + 50 * t) for i in range(each)]) for t in range(n)]
        got, failed = [[None] * each for _ in range(n)], []
        torch.cuda.synchronize()
        start = threading.Barrier(n)

        def work(t):
            try:
                stream = torch.cuda.Stream()
                start.wait(30)
                with torch.cuda.stream(stream):
                    for i, call in enumerate(calls[t]):
                        got[t][i] = call(stream)
                stream.synchronize()
            except BaseException as e:   # reported by the test's own thread
                failed.append(e)
        threads = [threading.Thread(target=work, args=(t,)) for t in range(n)]
        for t in threads:
            t.start()
        for t in threads:
            t.join(60)
        assert not failed, failed
        for t in range(n):
            for i in range(each):
                assert torch.equal(got[t][i], want[t][i]), (t, i)
    finally:
        torch.cuda.synchronize()
        gpu.sig_destroy(ctx)
        gpu.sig_destroy(calls_ctx)


def test_a_stream_that_is_gone_does_not_hold_the_context(gpu):
    """The last stream that used the scratch has been destroyed: the next call, on another one, still runs."""
    import torch
    hip = gpu.load()   # its dependencies resolve HIP's own entry points
    ctx = gpu.sig_create()
    try:
        calls = [scratch_call(gpu, ctx, i, 400) for i in range(2)]
        want = serial(calls)
        for i, call in enumerate(calls):
            handle = ctypes.c_void_p()
            assert hip.hipStreamCreate(ctypes.byref(handle)) == 0
            torch.cuda.synchronize()
            kept = call(handle.value)
            assert hip.hipStreamSynchronize(handle) == 0 and hip.hipStreamDestroy(handle) == 0
            got = call(torch.cuda.current_stream())
            torch.cuda.synchronize()
            assert torch.equal(got, want[i]) and torch.equal(kept, want[i])
    finally:
        torch.cuda.synchronize()
        gpu.sig_destroy(ctx)


def test_a_captured_call_survives_a_larger_one(gpu):
    """A graph keeps the address of the scratch it was captured with: an eager call that outgrows it leaves it in place."""
    import torch
    ctx = gpu.sig_create()
    try:
        x = torch.randn(4, 400, 5, device="cuda").cumsum(1) * 0.05
        large = torch.randn(512, 2000, 5, device="cuda").cumsum(1) * 0.02
        plan = gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, prefix_depth=2, chunks=4, segments=4)   # partial rows in scratch
        out = torch.empty((4, gpu.sig_size(5, 4)), device="cuda")
        assert gpu.sig_compute(ctx, x, 4, 0, out, plan=plan) == gpu.SIG_OK
        want = out.clone()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            assert gpu.sig_compute(ctx, x, 4, 0, out, plan=plan) == gpu.SIG_OK
        first = torch.empty((512, out.shape[1]), device="cuda")
        for _ in range(2):
            assert gpu.sig_compute(ctx, large, 4, 0, first, plan=plan) == gpu.SIG_OK   # 128 times the scratch
            taken = torch.full((1 << 20,), 7.0, device="cuda")
            out.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want) and bool((taken == 7.0).all())
    finally:
        torch.cuda.synchronize()
        gpu.sig_destroy(ctx)
