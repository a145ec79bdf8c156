"""Stream mode with the rows of a path split across workgroups (csrc/sig_split_rows.h), against the fp64 oracle with the gates of
test_gpu_parity.py, and the kernels that took these calls before (the same plan without it)."""
import numpy as np
import pytest

from paper_2501_08455_amd import workloads
from test_gpu_backward import launches
from test_gpu_parity import assert_parity, check, gpu, run_gpu  # noqa: F401
from test_gpu_stream_rows import _errors, assert_level1_is_added_up, copy_plan, infinite_points  # noqa: F401

pytestmark = pytest.mark.gpu

# d, depth, B, L, stretches a path: fewer steps than a block, ragged last blocks and stretches, stretches of one block, more stretches
# than the path has blocks; slices of whole wavefronts and ragged ones, one workgroup a path (many paths) and several (few)
CASES = [(10, 3, 3, 2, 1), (10, 3, 40, 20, 2), (8, 4, 2, 9, 1), (8, 4, 3, 10, 2), (8, 4, 1, 66, 7), (9, 4, 2, 18, 2), (9, 4, 1, 40, 5),
         (10, 4, 1, 33, 4), (10, 4, 2, 3, 1), (5, 5, 2, 50, 3), (5, 5, 3, 8, 1), (5, 5, 1, 300, 32), (6, 5, 1, 26, 3), (6, 5, 2, 9, 8),
         (4, 6, 2, 34, 4), (4, 6, 1, 17, 16), (10, 3, 300, 12, 1), (5, 5, 130, 10, 1), (6, 5, 70, 10, 1)]


@pytest.mark.parametrize("d,depth,B,L,segs", CASES)
def test_split_rows(gpu, oracle, d, depth, B, L, segs):  # noqa: F811
    x = workloads.brownian_paths(B, L, d, seed=9500 + 31 * d + 7 * depth + L + segs)
    plan = gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, split_rows=segs)
    check(gpu, oracle, x, depth, True, plan, label="split rows")


@pytest.mark.parametrize("d,depth,B,L", [(10, 4, 1, 400), (10, 4, 270, 20), (9, 4, 5, 90), (6, 5, 20, 70), (5, 5, 300, 30), (4, 6, 9, 200),
                                         (8, 4, 400, 90), (8, 4, 3, 400), (10, 3, 2000, 30)])
def test_planned_split_rows_agree_with_the_other_kernels(gpu, d, depth, B, L):  # noqa: F811
    rc, plan = gpu.sig_plan(gpu.default_ctx(), B, L, d, depth, 1)
    assert rc == gpu.SIG_OK and plan.split_rows >= 1, plan.as_dict()
    x = workloads.brownian_paths(B, L, d, seed=9600 + d + L)
    got = run_gpu(gpu, x, depth, True)
    assert np.array_equal(got, run_gpu(gpu, x, depth, True, plan))
    plan.split_rows = 0
    assert_parity(got, run_gpu(gpu, x, depth, True, plan).astype(np.float64), x, depth, True)


def test_split_rows_are_not_taken_where_they_do_not_apply(gpu):  # noqa: F811
    for d, depth, L, segs in [(7, 4, 50, 2), (2, 3, 50, 1), (10, 6, 9, 1), (8, 4, 50, 33), (8, 4, 5, 5), (9, 4, 50, -1)]:
        plan = gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, split_rows=segs)
        assert gpu.sig_plan_validate(2, L, d, depth, 1, plan) == gpu.SIG_ERR_INVALID
    assert gpu.sig_plan(None, 2, 60, 8, 4, 1)[1].split_rows == 0 and gpu.sig_plan(None, 2, 60, 10, 4, 0)[1].split_rows == 0


@pytest.mark.parametrize("d,depth,B,L,paths", [(10, 4, 2, 1500, 1), (10, 4, 40, 200, 4), (6, 5, 24, 500, 2), (5, 5, 64, 700, 4), (4, 6, 3, 900, 1),
                                               (8, 4, 300, 190, 8), (10, 3, 1800, 60, 64)])
def test_rounding_is_no_larger_than_the_other_kernels(gpu, oracle, d, depth, B, L, paths):  # noqa: F811
    """Both errors are means over hundreds of rows of thousands of coefficients: the ratio for equally accurate kernels is 1 +- 0.1."""
    rc, plan = gpu.sig_plan(gpu.default_ctx(), B, L, d, depth, 1)
    assert rc == gpu.SIG_OK and plan.split_rows >= 1
    x = workloads.brownian_paths(B, L, d, seed=9700 + d + L)
    split, other = _errors(gpu, oracle, x, depth, [plan, copy_plan(plan, split_rows=0)], paths)
    assert split <= 1.1 * other, (split, other)


@pytest.mark.parametrize("d,depth,B,L", [(10, 4, 2, 150), (10, 4, 140, 40), (6, 5, 2, 90), (8, 4, 3, 300), (10, 3, 1500, 20)])
def test_a_point_that_is_not_a_number_spoils_the_same_coefficients(gpu, d, depth, B, L):  # noqa: F811
    """Across a border of stretches too (first stretch, first step of another, last step)."""
    rc, plan = gpu.sig_plan(gpu.default_ctx(), B, L, d, depth, 1)
    assert rc == gpu.SIG_OK and plan.split_rows >= 1
    x = workloads.brownian_paths(B, L, d, seed=79)
    x[0, 5, 2] = np.nan
    x[1, (L - 1) // 2, d - 1] = np.nan
    x[B - 1, L - 1, 0] = np.nan
    got = np.isfinite(run_gpu(gpu, x, depth, True))
    plan.split_rows = 0
    assert np.array_equal(got, np.isfinite(run_gpu(gpu, x, depth, True, plan)))


@pytest.mark.parametrize("d,depth,B,L,segs", [(10, 3, 40, 40, 1), (10, 4, 8, 48, 3), (9, 4, 20, 40, 1), (6, 5, 9, 64, 4), (5, 5, 40, 40, 2), (4, 6, 25, 50, 3), (8, 4, 50, 50, 3)])
def test_infinite_points(gpu, d, depth, B, L, segs):  # noqa: F811
    """At the path's start, inside a block of steps and at its borders, at every border of stretches, and at the path's end."""
    rc, plan = gpu.sig_plan(gpu.default_ctx(), B, L, d, depth, 1)
    assert rc == gpu.SIG_OK
    sticky = plan.variant != gpu.SIG_VARIANT_LEVEL_SCAN or plan.row_workgroups > 0
    x = infinite_points(B, L, d, seed=89 + d, step=1 if B >= L else 8)
    plan.split_rows = segs
    got = run_gpu(gpu, x, depth, True, plan)
    plan.split_rows = 0
    assert_level1_is_added_up(x, got, run_gpu(gpu, x, depth, True, plan), sticky)


def test_without_scratch_what_lies_before_is_folded_again(gpu):  # noqa: F811
    """On a context without any, while a graph is recorded.  The entry point with fixed scratch has it: the same bits."""
    import torch
    x = workloads.brownian_paths(2, 700, 9, seed=81)
    xt = torch.from_numpy(x).cuda()
    want = run_gpu(gpu, x, 4, True)
    fresh = gpu.sig_create()
    out = torch.empty(want.shape, device="cuda")
    try:
        assert gpu.sig_plan(fresh, 2, 700, 9, 4, 1)[1].split_rows > 1
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            assert gpu.sig_compute(fresh, xt, 4, True, out) == gpu.SIG_OK
        for _ in range(3):
            out.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert_parity(out.cpu().numpy(), want.astype(np.float64), x, 4, True)
    finally:
        torch.cuda.synchronize()
        gpu.sig_destroy(fresh)
    out.fill_(float("nan"))
    assert gpu.sig_compute_noalloc(gpu.default_ctx(), xt, 4, 1, out) == gpu.SIG_OK   # 1.7 MB of the fixed scratch
    assert np.array_equal(out.cpu().numpy(), want)


@pytest.mark.parametrize("d,depth,B,L,most", [(4, 6, 20, 300, 1), (6, 5, 20, 300, 1), (9, 4, 2, 700, 2)])
def test_captured_calls_keep_off_scratch_that_their_plan_would_not_use(gpu, d, depth, B, L, most):  # noqa: F811
    """A graph of a call whose kernels without split rows take no scratch may run beside other calls: it holds one launch, on a context that
    has the scratch too.  (9,4), which goes launch by launch without split rows, holds two."""
    import torch
    ctx = gpu.sig_create()
    x = workloads.brownian_paths(B, L, d, seed=91)
    xt = torch.from_numpy(x).cuda()
    rc, plan = gpu.sig_plan(ctx, B, L, d, depth, 1)
    assert rc == gpu.SIG_OK and plan.split_rows > 1 and (plan.variant == gpu.SIG_VARIANT_LEVEL_SCAN and plan.row_workgroups == 0) == (most == 2)
    out = torch.empty((B, L - 1, gpu.sig_size(d, depth)), device="cuda")
    call = lambda: gpu.sig_compute(ctx, xt, depth, True, out)   # noqa: E731
    try:
        assert call() == gpu.SIG_OK            # the scratch grows here
        torch.cuda.synchronize()
        want = out.cpu().numpy()
        assert launches(gpu, call) == most
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            assert call() == gpu.SIG_OK
        for _ in range(3):
            out.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert_parity(out.cpu().numpy(), want.astype(np.float64), x, depth, True)
    finally:
        torch.cuda.synchronize()
        gpu.sig_destroy(ctx)
