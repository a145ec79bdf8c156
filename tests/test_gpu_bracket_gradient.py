"""The final-mode gradient swept on Lie brackets (csrc/sig_bracket.h) at the edges of its launches, against the fp64 oracle
with the gates of test_gpu_backward.py: several paths per wavefront with a ragged last one and a ragged last tile, chunks
side by side (chunk lengths with remainders, fewest steps, steps beyond the end), paths cut across workgroups, the
depth-2 kernel around its 256- and 512-point stretches, and the shortest paths that still come here."""
import numpy as np
import pytest

from paper_2501_08455_amd import workloads
from test_gpu_backward import check, gpu, launches, sampled_backward, say  # noqa: F401  (gpu is a fixture)

pytestmark = pytest.mark.gpu

# d, depth, B, L: batches that are packed (the oracle on the first, the last and a few in between)
PACKED = [(5, 4, 8197, 37), (5, 4, 20001, 18), (4, 4, 8200, 101), (2, 6, 16387, 33), (2, 3, 65541, 9), (3, 3, 20011, 64),
          (7, 4, 8195, 40), (8, 3, 8193, 13), (10, 3, 8193, 12), (3, 6, 9001, 35), (4, 5, 8191, 25)]


@pytest.mark.parametrize("case", PACKED, ids=lambda c: "-".join(str(v) for v in c))
def test_several_paths_per_wavefront(gpu, oracle, case):
    d, depth, B, L = case
    x = workloads.brownian_paths(B, L, d, seed=9000 + d + L)
    say("bracket gradient, packed: %s" % (case,))
    sampled_backward(gpu, oracle, x, depth, False, [0, 1, 7, B // 2, B - 3, B - 2, B - 1], seed=d + L)


# few paths: one workgroup per path and stretch of its steps
CUT = [(5, 4, 3, 101), (5, 4, 2, 102), (5, 4, 1, 17), (4, 4, 2, 500), (9, 4, 2, 12), (10, 4, 1, 43), (8, 4, 2, 12), (2, 4, 3, 14),
       (2, 4, 2, 259), (2, 3, 2, 2), (3, 3, 5, 5), (16, 3, 2, 50), (12, 3, 3, 401), (11, 3, 2, 3), (6, 5, 2, 500), (5, 5, 2, 26),
       (4, 6, 1, 90), (3, 6, 2, 700), (2, 6, 2, 1000), (2, 5, 3, 13), (6, 4, 1, 3001)]


@pytest.mark.parametrize("case", CUT, ids=lambda c: "-".join(str(v) for v in c))
def test_chunks_side_by_side(gpu, oracle, case):
    d, depth, B, L = case
    check(gpu, oracle, workloads.brownian_paths(B, L, d, seed=9100 + d + L), depth, False, seed=L, label="bracket, cut in time")


DEPTH2 = [(2, 3, 2), (2, 300, 3), (3, 700, 100), (5, 2, 255), (5, 2, 256), (5, 3, 257), (20, 2, 513), (17, 1, 300), (13, 5, 3), (11, 90, 40)]


@pytest.mark.parametrize("d,B,L", DEPTH2)
def test_depth_two(gpu, oracle, d, B, L):
    check(gpu, oracle, workloads.brownian_paths(B, L, d, seed=9200 + d + L), 2, False, seed=L, label="bracket, depth 2")


# ||gpu - oracle||_F / ||oracle||_F of a batch: four times the largest of 522 settings (29 shapes, 16 to 2,000 points; Brownian,
# drifting, uniform, unscaled and zigzag paths) per depth: 1.5e-7, 2.0e-7, 5.7e-7, 1.1e-6, 1.6e-6.  The sweep on signatures
# was at 1.0 to 50 times these errors, so that a sum held too short or a bracket value lost would show.
ROUNDING = {2: 6e-7, 3: 8e-7, 4: 2.3e-6, 5: 4.4e-6, 6: 6.4e-6}


@pytest.mark.parametrize("scaled", [True, False], ids=["scaled", "unscaled"])
@pytest.mark.parametrize("d,depth,B,L", [(3, 2, 32, 400), (20, 2, 32, 100), (2, 3, 32, 2000), (16, 3, 16, 400), (5, 4, 32, 100),
                                         (10, 4, 3, 2000), (4, 4, 9000, 60), (2, 5, 32, 400), (6, 5, 4, 400), (2, 6, 32, 2000),
                                         (4, 6, 8, 100)])
def test_errors_stay_at_the_rounding_of_float32(gpu, oracle, d, depth, B, L, scaled):
    import torch
    rng = np.random.default_rng(9500 + d + L)
    x = (rng.normal(size=(B, L, d)) * (L ** -0.5 if scaled else 1.0)).cumsum(1).astype(np.float32)
    path = torch.from_numpy(x).cuda()
    out = gpu.signature(path, depth)
    g = torch.from_numpy(rng.normal(size=tuple(out.shape)).astype(np.float32)).cuda()
    gx = torch.full_like(path, float("nan"))
    assert gpu.sig_backward(gpu.default_ctx(), path, depth, 0, out, g, gx) == gpu.SIG_OK
    pick = np.unique(np.linspace(0, B - 1, 32).astype(int))
    got = gx[torch.from_numpy(pick).cuda()].cpu().numpy().astype(np.float64)
    want = oracle.signature_backward(x[pick], depth, g.cpu().numpy()[pick])
    err = np.linalg.norm(got - want) / np.linalg.norm(want)
    say("  rel err %.2e (gate %.1e)" % (err, ROUNDING[depth]))
    assert err <= ROUNDING[depth]


# d, depth, paths, points: the last length on signatures and the first on brackets, where the batch moves that point
BORDERS = [(3, 2, 64, 3), (5, 2, 300, 5), (10, 2, 64, 10), (10, 2, 63, 3), (8, 2, 5000, 6), (8, 2, 17000, 7), (5, 2, 66000, 5), (2, 3, 600, 17), (2, 3, 1500, 21),
           (2, 3, 100, 13), (2, 3, 16400, 7), (3, 3, 700, 12), (4, 3, 66000, 9), (4, 3, 40, 8), (5, 3, 600, 8), (5, 3, 66000, 9),
           (6, 3, 16500, 13), (7, 3, 16500, 13), (7, 3, 66000, 17), (7, 3, 30, 5), (8, 3, 100, 12), (8, 3, 4100, 8), (9, 3, 100, 10),
           (10, 3, 1100, 6), (2, 4, 600, 17), (2, 4, 1100, 25), (2, 4, 9, 13), (4, 4, 4200, 17), (3, 5, 1100, 17), (3, 5, 5000, 20),
           (9, 4, 20, 13), (10, 4, 20, 16), (5, 5, 1100, 25)]


@pytest.mark.parametrize("d,depth,B,L", BORDERS)
def test_both_sides_of_the_shortest_path_on_brackets(gpu, oracle, d, depth, B, L):
    import torch
    for points in (L - 1, L):
        x = workloads.brownian_paths(B, points, d, seed=9600 + d + points)
        say("short paths: (%d,%d) %d paths of %d points" % (d, depth, B, points))
        sampled_backward(gpu, oracle, x, depth, False, sorted({0, 1, B // 2, B - 2, B - 1}), seed=d + points)
        path = torch.from_numpy(x).cuda()   # a fresh context: the sweeps that need no scratch, brackets in place of the others
        out, ctx = gpu.signature(path, depth), gpu.sig_create()
        g, gx = torch.ones_like(out), torch.empty_like(path)
        try:
            assert launches(gpu, lambda: gpu.sig_backward(ctx, path, depth, 0, out, g, gx)) == 1
        finally:
            torch.cuda.synchronize()
            gpu.sig_destroy(ctx)


# few long paths at depth 5 and 6: what lies behind a stretch is folded by more slots than the workgroup has chunks
BEHIND = [(6, 5, 1, 600), (6, 5, 2, 2000), (6, 5, 1, 2011), (6, 5, 20, 800), (5, 5, 1, 1500), (5, 5, 3, 777), (4, 5, 1, 2000), (4, 5, 2, 901),
          (4, 6, 1, 1200), (4, 6, 3, 333), (3, 6, 1, 2000), (2, 6, 1, 5003), (3, 5, 1, 4000)]


@pytest.mark.parametrize("d,depth,B,L", BEHIND)
def test_long_paths_cut_across_workgroups(gpu, oracle, d, depth, B, L):
    assert gpu.sig_backward_segments(None, B, L, d, depth, 0) > 1
    x = workloads.brownian_paths(B, L, d, seed=9650 + L)
    a = check(gpu, oracle, x[:3], depth, False, seed=L, label="what lies behind")
    np.testing.assert_array_equal(a, check(gpu, oracle, x[:3], depth, False, seed=L, label="again"))


def test_the_gradient_of_a_translation_vanishes(gpu):
    """The signature does not see where a path starts: the gradients of a path's points add up to zero, up to the rounding
    of 2,000 sums of float32 values (the sum of their magnitudes times 2^-23)."""
    import torch
    x = torch.from_numpy(workloads.brownian_paths(64, 2000, 5, seed=9300)).cuda()
    out = gpu.signature(x, 4)
    g = torch.randn_like(out)
    gx = torch.full_like(x, float("nan"))
    assert gpu.sig_backward(gpu.default_ctx(), x, 4, 0, out, g, gx) == gpu.SIG_OK
    total, size = gx.double().sum(1), gx.double().abs().sum(1)
    worst = float((total.abs() / size).max())
    say("sum of a path's gradients over the sum of their magnitudes: %.1e" % worst)
    assert np.isfinite(worst) and worst <= 2.0 ** -18


@pytest.mark.parametrize("d,depth,B,L", [(5, 4, 128, 100), (5, 4, 8200, 40), (10, 4, 2, 900), (12, 3, 93, 50), (20, 2, 7, 600),
                                         (4, 6, 2, 90), (6, 5, 128, 500)])
def test_one_launch_and_no_scratch(gpu, d, depth, B, L):
    """What tells the sweep on brackets from the others: a context that has no scratch gets none, under capture too."""
    import torch
    x = torch.from_numpy(workloads.brownian_paths(B, L, d, seed=9400 + L)).cuda()
    out = gpu.signature(x, depth)
    g, gx = torch.randn_like(out), torch.empty_like(x)
    ctx = gpu.sig_create()
    try:
        assert launches(gpu, lambda: gpu.sig_backward(ctx, x, depth, 0, out, g, gx)) == 1
    finally:
        torch.cuda.synchronize()
        gpu.sig_destroy(ctx)
