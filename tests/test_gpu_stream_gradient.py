"""The every-prefix gradient at depth 2 and, for 11 and 12 channels, 3 (csrc/sig_stream_gradient.hip) at the edges of its launches, against the fp64 oracle with
the gates of test_gpu_backward.py: fewer rows than a tile, ragged last tiles, stretches, blocks and workgroups, whole paths side by
side with a ragged last wavefront, every channel count; and without scratch, as a captured call may have to run."""
import numpy as np
import pytest

from paper_2501_08455_amd import workloads
from test_gpu_backward import check, gpu, launches, sampled_backward, say  # noqa: F401  (gpu is a fixture)

pytestmark = pytest.mark.gpu

# d, B, L: a stretch per slot (several paths in a workgroup, or one), several blocks of a workgroup, several workgroups a path
CUT = [(2, 3, 2), (2, 5, 130), (3, 2, 85), (5, 3, 9), (6, 1, 4), (9, 4, 2), (10, 3, 26), (13, 2, 17), (17, 2, 13), (20, 5, 60),
       (16, 128, 40), (20, 300, 70), (2, 40, 1025), (9, 300, 1300), (18, 300, 301),
       (10, 1, 1445), (4, 2, 3001), (19, 1, 700), (12, 3, 501)]


@pytest.mark.parametrize("d,B,L", CUT)
def test_stretches_side_by_side(gpu, oracle, d, B, L):
    x = workloads.brownian_paths(B, L, d, seed=9600 + d + L)
    say("every-prefix gradient, depth 2, cut in time: %s" % ((d, B, L),))
    sampled_backward(gpu, oracle, x, 2, True, sorted({0, B // 2, B - 1}), seed=d + L)


# whole paths side by side: more of them than a wavefront holds, and rows that are no multiple of a tile
@pytest.mark.parametrize("d,B,L", [(2, 40001, 3), (2, 9001, 34), (3, 22003, 2), (5, 13001, 12), (7, 9002, 31), (10, 8193, 9), (16, 4099, 5),
                                   (20, 3001, 8), (13, 4501, 3)])
def test_whole_paths_side_by_side(gpu, oracle, d, B, L):
    x = workloads.brownian_paths(B, L, d, seed=9700 + d + L)
    say("every-prefix gradient, depth 2, uncut: %s" % ((d, B, L),))
    sampled_backward(gpu, oracle, x, 2, True, [0, 1, B // 2, B - 2, B - 1], seed=d + L)


# depth 3: fewer rows than a tile, odd numbers of them, several paths in a workgroup, blocks, workgroups a path (few paths), uncut
@pytest.mark.parametrize("d,B,L", [(11, 1, 2), (12, 3, 2), (11, 2, 3), (12, 5, 4), (11, 300, 4), (12, 46, 71), (11, 9, 96), (12, 1, 300), (11, 260, 60),
                                   (12, 270, 41), (11, 8200, 3), (12, 8195, 4)])
def test_depth_three(gpu, oracle, d, B, L):
    x = workloads.brownian_paths(B, L, d, seed=9750 + d + L)
    say("every-prefix gradient, depth 3: %s" % ((d, B, L),))
    sampled_backward(gpu, oracle, x, 3, True, sorted({0, B // 2, B - 1}), seed=d + L)


@pytest.mark.parametrize("d,L", [(11, 121), (12, 121), (12, 700)])
def test_errors_at_depth_three_stay_at_the_rounding_of_float32(gpu, oracle, d, L):
    """As below: u sqrt(K) of the norm, measured 1.6e-7 to 2.4e-7."""
    import torch
    rng = np.random.default_rng(9850 + d)
    x = (rng.normal(size=(3, L, d)) * L ** -0.5).cumsum(1).astype(np.float32)
    path = torch.from_numpy(x).cuda()
    out = gpu.signature(path, 3, stream=True)
    g = torch.from_numpy(rng.normal(size=tuple(out.shape)).astype(np.float32)).cuda()
    gx = torch.full_like(path, float("nan"))
    assert gpu.sig_backward(gpu.default_ctx(), path, 3, 1, out, g, gx) == gpu.SIG_OK
    want = oracle.signature_backward(x, 3, g.cpu().numpy(), stream=True)
    err = np.linalg.norm(gx.cpu().numpy() - want) / np.linalg.norm(want)
    say("  d = %d, L = %d: rel err %.2e" % (d, L, err))
    assert err <= 2.0 ** -24 * (L - 1) ** 0.5


@pytest.mark.parametrize("d", range(2, 21))
def test_errors_stay_at_the_rounding_of_float32(gpu, oracle, d):
    """A row's point is a sum of K terms of the rows behind it: u sqrt(K) = 6.6e-7 of its norm for K = 120 at worst, measured
    1.7e-7 at most."""
    import torch
    rng = np.random.default_rng(9800 + d)
    x = (rng.normal(size=(5, 121, d)) * 121 ** -0.5).cumsum(1).astype(np.float32)
    path = torch.from_numpy(x).cuda()
    out = gpu.signature(path, 2, stream=True)
    g = torch.from_numpy(rng.normal(size=tuple(out.shape)).astype(np.float32)).cuda()
    gx = torch.full_like(path, float("nan"))
    assert gpu.sig_backward(gpu.default_ctx(), path, 2, 1, out, g, gx) == gpu.SIG_OK
    want = oracle.signature_backward(x, 2, g.cpu().numpy(), stream=True)
    err = np.linalg.norm(gx.cpu().numpy() - want) / np.linalg.norm(want)
    say("  d = %d: rel err %.2e" % (d, err))
    assert err <= 6.6e-7


def test_a_capture_that_cannot_grow_scratch_keeps_a_path_in_one_workgroup(gpu, oracle):
    """One long path takes two launches and scratch; on a context without any, while a graph is recorded, one launch."""
    import torch
    x = workloads.brownian_paths(1, 1500, 6, seed=9900)
    xt = torch.from_numpy(x).cuda()
    out = gpu.signature(xt, 2, stream=True)
    g = torch.from_numpy(np.random.default_rng(5).normal(size=tuple(out.shape)).astype(np.float32)).cuda()
    want = oracle.signature_backward(x, 2, g.cpu().numpy(), stream=True)
    fresh, gx = gpu.sig_create(), torch.empty_like(xt)
    call = lambda ctx: gpu.sig_backward(ctx, xt, 2, 1, out, g, gx)   # noqa: E731
    try:
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            assert call(fresh) == gpu.SIG_OK
        for _ in range(3):
            gx.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert np.linalg.norm(gx.cpu().numpy() - want) <= 1e-5 * np.linalg.norm(want)
        assert launches(gpu, lambda: call(fresh)) == 1
        assert call(fresh) == gpu.SIG_OK            # the scratch grows here
        assert launches(gpu, lambda: call(fresh)) == 2
    finally:
        torch.cuda.synchronize()
        gpu.sig_destroy(fresh)


@pytest.mark.parametrize("d,B,L,most", [(6, 3, 400, 1), (10, 60, 700, 1), (6, 3, 900, 2), (15, 3, 200, 2)])
def test_captured_calls_share_scratch_only_for_few_long_paths(gpu, oracle, d, B, L, most):
    """A graph may run beside other calls of the context: it holds one launch also where the scratch is there, but for calls that any sweep
    cuts with scratch."""
    import torch
    x = workloads.brownian_paths(B, L, d, seed=9905 + d)
    xt = torch.from_numpy(x).cuda()
    out = gpu.signature(xt, 2, stream=True)
    g = torch.from_numpy(np.random.default_rng(6).normal(size=tuple(out.shape)).astype(np.float32)).cuda()
    ctx, gx = gpu.sig_create(), torch.empty_like(xt)
    call = lambda: gpu.sig_backward(ctx, xt, 2, 1, out, g, gx)   # noqa: E731
    try:
        assert gpu.sig_backward_segments(ctx, B, L, d, 2, 1) > 1 and call() == gpu.SIG_OK      # the scratch grows here
        assert launches(gpu, call) == most
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            assert call() == gpu.SIG_OK
        pick = sorted({0, B - 1})
        want = oracle.signature_backward(x[pick], 2, g[pick].cpu().numpy(), stream=True)
        for _ in range(3):
            gx.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert np.linalg.norm(gx[pick].cpu().numpy() - want) <= 1e-5 * np.linalg.norm(want)
    finally:
        torch.cuda.synchronize()
        gpu.sig_destroy(ctx)


def test_depth_three_without_enough_scratch_takes_the_general_sweep(gpu, oracle):
    """A capture on a context whose scratch holds what the general sweep needs, but not the reduced rows."""
    import torch
    x = workloads.brownian_paths(2, 40, 12, seed=9910)
    xt = torch.from_numpy(x).cuda()
    out = gpu.signature(xt, 3, stream=True)
    g = torch.from_numpy(np.random.default_rng(6).normal(size=tuple(out.shape)).astype(np.float32)).cuda()
    want = oracle.signature_backward(x, 3, g.cpu().numpy(), stream=True)
    fresh, gx = gpu.sig_create(), torch.empty_like(xt)
    call = lambda: gpu.sig_backward(fresh, xt, 3, 1, out, g, gx)   # noqa: E731
    try:
        small = torch.from_numpy(workloads.brownian_paths(8, 14, 13, seed=3)).cuda()     # the general sweep of (13,3): 8 x 13 x 13 floats and more
        rows = gpu.signature(small, 3, stream=True)
        assert gpu.sig_backward(fresh, small, 3, 1, rows, torch.ones_like(rows), torch.empty_like(small)) == gpu.SIG_OK
        general = launches(gpu, call)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            assert call() == gpu.SIG_OK
        for _ in range(3):
            gx.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert np.linalg.norm(gx.cpu().numpy() - want) <= 1e-5 * np.linalg.norm(want)
        assert call() == gpu.SIG_OK                 # the scratch grows here
        assert launches(gpu, call) != general
    finally:
        torch.cuda.synchronize()
        gpu.sig_destroy(fresh)


def test_rows_of_more_floats_than_32_bits_count(gpu):
    """One path whose rows take 2^31 floats and more: workgroups count from their own first row.  Upstream gradients in a few rows
    only, at the borders of stretches and workgroups among them, so that float64 gives the gradient of every point: products of twenty
    terms, a few roundings each."""
    import torch
    d, L = 20, 5_200_000
    K, D = L - 1, d + d * d
    assert K * D > 2 ** 31 and gpu.sig_backward_segments(None, 1, L, d, 2, 1) > 1
    gen = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn((1, L, d), device="cuda", generator=gen)
    g = torch.zeros((1, K, D), device="cuda")
    W = gpu.sig_backward_segments(None, 1, L, d, 2, 1)
    rows = sorted({0, 1, K // 3, K - 1} | {K // W * w + o for w in (1, 2, W - 1) for o in range(-40, 41, 8)})
    g[0, rows] = torch.randn((len(rows), D), device="cuda", generator=gen)
    gx = torch.full_like(x, float("nan"))
    assert gpu.sig_backward(gpu.default_ctx(), x, 2, 1, g, g, gx) == gpu.SIG_OK      # (the rows of S are not read)
    X, G = x[0].double(), g[0, rows].double()
    del g
    M = G[:, d:].reshape(-1, d, d)
    sums = torch.cat([(M - M.transpose(1, 2)).flip(0).cumsum(0).flip(0), torch.zeros_like(M[:1])])   # A of the rows up to each of `rows`
    v = X[1:] - X[:-1]
    half = torch.empty_like(v)                         # half of sum_a v[a] A[a b]
    at = [0] + [r + 1 for r in rows] + [K]
    for i in range(len(at) - 1):
        half[at[i]:at[i + 1]] = 0.5 * v[at[i]:at[i + 1]] @ sums[i]
    want = torch.zeros_like(X)
    want[1:] -= half
    want[:-1] -= half
    S = X[[r + 1 for r in rows]] - X[0]
    want[[r + 1 for r in rows]] += G[:, :d] + (S.unsqueeze(2) * M).sum(1)
    want[0] -= (G[:, :d] + (M * S.unsqueeze(1)).sum(2)).sum(0)
    err = float((gx[0].double() - want).norm() / want.norm())
    say("  %d rows of %d floats: rel err %.2e" % (K, D, err))
    assert bool(torch.isfinite(gx).all()) and err <= 1e-6
