"""Stream mode with the rows written straight from registers and the paths cut across workgroups (csrc/sig_stream_rows.h),
against the fp64 oracle with the gates of test_gpu_parity.py, and the general route (the same plan without it)."""
import numpy as np
import pytest

from paper_2501_08455_amd import workloads
from test_gpu_parity import assert_parity, check, gpu, run_gpu  # noqa: F401

pytestmark = pytest.mark.gpu

# d, depth, B, L, workgroups a path is cut across.  Slots of 8 lanes (eight to a wavefront) to 512 (eight wavefronts), whole
# wavefronts and ragged ones; one piece or many; the shortest paths; pieces and workgroups left without steps; tiles that do not
# hold a piece (one piece of 300 steps of (20,2)) nor what lies before it
CASES = [
    (2, 4, 3, 2, 1), (2, 4, 3, 3, 2), (2, 4, 5, 40, 1), (2, 4, 2, 257, 5), (3, 3, 7, 25, 1), (3, 3, 2, 90, 3), (4, 3, 3, 130, 4),
    (8, 2, 4, 64, 1), (9, 2, 3, 200, 6), (10, 2, 2, 333, 2), (11, 2, 5, 33, 1), (16, 2, 3, 100, 4), (20, 2, 2, 301, 1),
    (20, 2, 1, 1500, 2), (5, 3, 3, 99, 32), (8, 3, 2, 100, 3), (10, 3, 2, 75, 2), (11, 3, 2, 50, 2), (12, 3, 2, 61, 4),
    (4, 4, 3, 256, 4), (4, 4, 1, 2, 1), (4, 4, 2, 700, 7), (5, 4, 2, 100, 16), (6, 4, 2, 60, 3), (7, 4, 1, 50, 2), (8, 4, 1, 40, 3),
    (2, 5, 3, 70, 2), (3, 5, 2, 80, 3), (4, 5, 1, 60, 4), (2, 6, 2, 300, 3), (3, 6, 1, 50, 2),
]


@pytest.mark.parametrize("d,depth,B,L,segs", CASES)
def test_rows_from_registers(gpu, oracle, d, depth, B, L, segs):  # noqa: F811
    x = workloads.brownian_paths(B, L, d, seed=9100 + 31 * d + 7 * depth + L + segs)
    plan = gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, row_workgroups=segs)
    check(gpu, oracle, x, depth, True, plan, label="rows")


def copy_plan(plan, **fields):
    other = type(plan).from_buffer_copy(plan)
    for name, value in fields.items():
        setattr(other, name, value)
    return other


def rows_plan(plan):
    """The plan's rows from registers, as they run where no split_rows come before them."""
    assert plan.row_workgroups >= 1
    return copy_plan(plan, split_rows=0)


def other_plan(plan):
    """... and its register or level kernels."""
    return copy_plan(plan, split_rows=0, row_workgroups=0)


@pytest.mark.parametrize("d,depth,B,L", [(4, 4, 64, 256), (5, 4, 16, 100), (3, 4, 300, 57), (16, 2, 1500, 40), (13, 2, 1027, 23),
                                         (12, 3, 40, 90), (10, 3, 4, 700), (2, 6, 1025, 30), (20, 2, 5, 5000)])
def test_planned_rows_agree_with_the_other_kernels(gpu, oracle, d, depth, B, L):  # noqa: F811
    """The planner's own cut, whole paths side by side in a workgroup included, against the plan's other kernels: no row
    further apart than two foldings of the same increments can be (assert_parity's bounds, on every row).  (At depth 2 the plan
    comes with rows that need no scan, which are taken off it.)"""
    rc, plan = gpu.sig_plan(gpu.default_ctx(), B, L, d, depth, 1)
    assert rc == gpu.SIG_OK and plan.row_workgroups >= 1, plan.as_dict()
    x = workloads.brownian_paths(B, L, d, seed=9300 + d + L)
    if plan.split_rows == 0:
        assert np.array_equal(run_gpu(gpu, x, depth, True), run_gpu(gpu, x, depth, True, plan))
    rows, other = rows_plan(plan), other_plan(plan)
    got = run_gpu(gpu, x, depth, True, rows)
    assert_parity(got, run_gpu(gpu, x, depth, True, other).astype(np.float64), x, depth, True)


def test_a_point_that_is_not_a_number_spoils_the_same_coefficients(gpu):  # noqa: F811
    x = workloads.brownian_paths(2, 120, 4, seed=77)
    x[0, 71, 2] = np.nan
    other = np.isfinite(run_gpu(gpu, x, 4, True, gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, prefix_depth=2)))
    assert other[0, :70].all() and not other[0, 70:, 2].any()
    for segs in (1, 4, 9):
        got = run_gpu(gpu, x, 4, True, gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, row_workgroups=segs))
        assert np.array_equal(np.isfinite(got), other)


def infinite_points(B, L, d, seed, first=0, step=1):
    """Paths with one infinite point each, of either sign: path b's is point (first + b * step) % L."""
    x = workloads.brownian_paths(B, L, d, seed=seed)
    for b in range(B):
        x[b, (first + b * step) % L, b % d] = np.inf if b % 3 else -np.inf
    return x


def assert_level1_is_added_up(x, got, other, sticky=True):
    """Level 1 is infinite or NaN where the sum of the increments is (or, not sticky, the distance from the first point), with the
    same sign; the other kernels agree, and on which coefficients of the other levels are finite."""
    d = x.shape[-1]
    with np.errstate(invalid="ignore"):
        want = np.diff(x.astype(np.float64), axis=1).cumsum(1) if sticky else x[:, 1:] - x[:, :1]
    for rows in (got, other):
        for kind in (np.isnan, np.isposinf, np.isneginf):
            assert np.array_equal(kind(rows[..., :d]), kind(want))
    assert np.array_equal(np.isfinite(got), np.isfinite(other))


@pytest.mark.parametrize("d,depth,B,L,segs", [(4, 4, 64, 50, 1), (4, 4, 90, 90, 4), (8, 2, 70, 70, 3), (5, 3, 60, 60, 5), (10, 3, 40, 40, 2),
                                              (12, 2, 60, 60, 2), (11, 3, 30, 30, 1)])
def test_infinite_points(gpu, d, depth, B, L, segs):  # noqa: F811
    """At the path's start, at every border of pieces and workgroups, and at its end."""
    x = infinite_points(B, L, d, seed=85 + d)
    got = run_gpu(gpu, x, depth, True, gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, row_workgroups=segs))
    rc, plan = gpu.sig_plan(gpu.default_ctx(), B, L, d, depth, 1)
    plan.row_workgroups = plan.split_rows = 0
    assert_level1_is_added_up(x, got, run_gpu(gpu, x, depth, True, plan), sticky=d <= 10)


def test_rows_are_not_taken_where_they_do_not_apply(gpu):  # noqa: F811
    for d, depth, L, segs in [(4, 6, 50, 2), (2, 3, 50, 1), (4, 4, 50, 33), (4, 4, 5, 5), (13, 3, 20, 1)]:
        plan = gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, row_workgroups=segs)
        assert gpu.sig_plan_validate(2, L, d, depth, 1, plan) == gpu.SIG_ERR_INVALID
    assert gpu.sig_plan(None, 4096, 256, 4, 4, 1)[1].row_workgroups == 0
    assert gpu.sig_plan(None, 64, 256, 4, 4, 0)[1].row_workgroups == 0


def _errors(gpu, oracle, x, depth, plans, paths):
    """Relative error of each plan against the fp64 oracle, over the first `paths` paths.  The plans name different kernels."""
    import torch
    named = {(p.split_rows > 0, p.split_rows == 0 and p.row_workgroups > 0) for p in plans}
    assert len(named) == len(plans), [p.as_dict() for p in plans]
    want = oracle.signature(x[:paths].astype(np.float64), depth, stream=True)
    xt = torch.from_numpy(x).cuda()
    errs = []
    for plan in plans:
        out = torch.empty((x.shape[0], x.shape[1] - 1, want.shape[-1]), device="cuda")
        assert gpu.sig_compute(gpu.default_ctx(), xt, depth, True, out, plan=plan) == gpu.SIG_OK
        got = out[:paths].cpu().numpy().astype(np.float64)
        del out
        errs.append(np.linalg.norm(got - want) / np.linalg.norm(want))
    return errs


@pytest.mark.parametrize("d,depth,B,L,paths", [(12, 3, 130, 1000, 8), (11, 3, 130, 1500, 8), (20, 2, 130, 2000, 16), (17, 2, 200, 1500, 16),
                                               (2, 5, 1100, 900, 64), (2, 6, 300, 1500, 64), (3, 5, 300, 290, 32), (12, 2, 64, 12, 64), (16, 2, 9, 20, 9)])
def test_rounding_is_no_larger_than_the_other_kernels(gpu, oracle, d, depth, B, L, paths):  # noqa: F811
    """Long pieces, and short paths whose level 1 dominates.  Both errors are means over thousands of rows of `paths` independent
    paths; the ratio of two such means of equally accurate kernels stays within 1 +- 0.1 (with plain sums over the whole piece and
    level 1 added up, every case here lies beyond)."""
    rc, plan = gpu.sig_plan(gpu.default_ctx(), B, L, d, depth, 1)
    assert rc == gpu.SIG_OK and plan.row_workgroups >= 1
    x = workloads.brownian_paths(B, L, d, seed=9400 + d + L)
    if L < 30:   # uniform increments: level 1 is not small against the others
        x = workloads.uniform_paths(B, L, d, seed=9401 + d)
    rows, other = _errors(gpu, oracle, x, depth, [rows_plan(plan), other_plan(plan)], paths)
    assert rows <= 1.1 * other, (rows, other)


@pytest.mark.parametrize("d,depth,L,segs", [(12, 2, 14, 1), (12, 2, 300, 3), (20, 2, 500, 1), (16, 2, 900, 5), (11, 3, 120, 2), (12, 3, 700, 1)])
def test_level_1_of_many_channels_comes_from_the_points(gpu, d, depth, L, segs):  # noqa: F811
    """Points that are not numbers, at a piece's first step too, spoil the same coefficients as in the launches per level: level 1
    is finite again in the next row."""
    x = workloads.brownian_paths(3, L, d, seed=78)
    x[0, L // 2, 2] = np.nan
    x[1, 1, d - 1] = np.inf
    x[2, L - 2, 0] = np.nan
    got = run_gpu(gpu, x, depth, True, gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, row_workgroups=segs))
    want = run_gpu(gpu, x, depth, True, gpu.make_plan(gpu.SIG_VARIANT_LEVEL_SCAN, chunks=0))
    assert np.array_equal(np.isfinite(got), np.isfinite(want))
    assert np.isfinite(got[0, L // 2:, :d]).all() and not np.isfinite(got[0, L // 2 - 1, 2])
    ok = np.isfinite(want[:, :, :d])
    assert np.array_equal(got[:, :, :d][ok], want[:, :, :d][ok])   # one difference each: the same bits
