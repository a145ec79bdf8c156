"""Stream mode at depth 2 (csrc/sig_depth2_rows.hip): whole paths side by side, stretches of a path side by side, and paths across
workgroups, against the fp64 oracle with the gates of test_gpu_parity.py and the kernels that took these calls before."""
import numpy as np
import pytest

from paper_2501_08455_amd import workloads
from test_gpu_parity import assert_parity, check, gpu, run_gpu  # noqa: F401
from test_gpu_stream_rows import _errors, assert_level1_is_added_up, copy_plan, infinite_points  # noqa: F401

pytestmark = pytest.mark.gpu

# d, B, L, workgroups a path: one step; a tile of steps and one more or less; one path more or less than a wavefront's slots and a
# workgroup's; a stretch of one step; stretches that end before the path does; a last workgroup with fewer stretches than slots
CASES = [(2, 1, 2, 1), (2, 33, 17, 1), (2, 31, 18, 1), (2, 3, 40, 1), (2, 2, 300, 2), (2, 1, 77, 32), (3, 21, 16, 1), (3, 5, 32, 1), (3, 2, 66, 3),
         (4, 17, 20, 1), (4, 2, 530, 8), (5, 12, 9, 1), (5, 13, 34, 1), (6, 11, 7, 1), (6, 1, 201, 5), (7, 9, 33, 1), (8, 8, 12, 1), (8, 9, 65, 2),
         (9, 8, 14, 1), (10, 7, 31, 1), (10, 2, 100, 7), (11, 6, 11, 1), (11, 5, 45, 1), (12, 5, 32, 1), (12, 6, 33, 1), (13, 4, 70, 4), (14, 5, 30, 1),
         (15, 4, 35, 1), (16, 5, 6, 1), (16, 16, 33, 1), (16, 17, 40, 1), (17, 3, 64, 9), (18, 4, 33, 1), (19, 3, 5, 1), (19, 13, 50, 1), (20, 4, 4, 1),
         (20, 1, 333, 16), (20, 2, 5, 4), (14, 16, 81, 1), (15, 2, 130, 2), (17, 12, 70, 1), (20, 2, 400, 2)]


@pytest.mark.parametrize("d,B,L,segs", CASES)
def test_depth2_rows(gpu, oracle, d, B, L, segs):  # noqa: F811
    x = workloads.brownian_paths(B, L, d, seed=9800 + 31 * d + L + segs)
    check(gpu, oracle, x, 2, True, gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, split_rows=segs), label="depth 2 rows")


# d, B, L, whole paths (as many workgroups of 64 / d paths as that takes)
PLANNED = [(2, 60003, 60, True), (3, 40001, 130, True), (4, 30000, 90, True), (5, 300, 70, False), (6, 3, 900, False), (7, 20, 400, False),
           (8, 1000, 150, False), (9, 100, 80, False), (10, 60, 200, False), (11, 40000, 5, True), (13, 1027, 33, False), (16, 1500, 40, False),
           (20, 5, 5000, False), (20, 20001, 6, True)]


@pytest.mark.parametrize("d,B,L,whole", PLANNED)
def test_planned_depth2_rows_agree_with_the_other_kernels(gpu, d, B, L, whole):  # noqa: F811
    """The other kernels with each other too: the plan's register or level kernel, and the rows of csrc/sig_stream_rows.h."""
    rc, plan = gpu.sig_plan(gpu.default_ctx(), B, L, d, 2, 1)
    assert rc == gpu.SIG_OK and plan.split_rows >= 1, plan.as_dict()
    rc, _, workgroups, scratch = gpu.sig_plan_footprint(B, L, d, 2, 1, plan)
    assert rc == gpu.SIG_OK and scratch == 0 and (workgroups == -(-B // (64 // d))) == whole
    x = workloads.brownian_paths(B, L, d, seed=9850 + d + L)
    got = run_gpu(gpu, x, 2, True)
    assert np.array_equal(got, run_gpu(gpu, x, 2, True, plan))
    plan.split_rows = 0
    if plan.row_workgroups > 0:
        assert_parity(got, run_gpu(gpu, x, 2, True, plan).astype(np.float64), x, 2, True)
        plan.row_workgroups = 0
    assert_parity(got, run_gpu(gpu, x, 2, True, plan).astype(np.float64), x, 2, True)


def test_depth2_rows_are_not_taken_where_they_do_not_apply(gpu):  # noqa: F811
    for d, L, segs in [(1, 50, 1), (21, 50, 1), (4, 50, 33), (4, 5, 5), (4, 50, -1), (20, 6000000, 1)]:
        plan = gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, split_rows=segs)
        assert gpu.sig_plan_validate(2, L, d, 2, 1, plan) == gpu.SIG_ERR_INVALID
    for B, L, d in [(64, 20, 12), (64, 40, 4), (600, 900, 2), (5, 10 ** 7, 20)]:
        assert gpu.sig_plan(None, B, L, d, 2, 1)[1].split_rows == 0
    assert gpu.sig_plan(None, 60, 200, 10, 2, 0)[1].split_rows == 0


@pytest.mark.parametrize("d,B,L,paths", [(2, 30003, 200, 40), (4, 2, 1500, 2), (5, 300, 170, 16), (8, 1000, 150, 10), (10, 3, 1200, 3), (12, 600, 300, 8),
                                         (13, 8000, 40, 20), (20, 5, 2000, 1)])
def test_rounding_is_no_larger_than_the_other_kernels(gpu, oracle, d, B, L, paths):  # noqa: F811
    """The kernels that the rest of the plan names: register kernels, and for (10,2), (12,2), (13,2) and (20,2) rows from registers.
    Both errors are means over hundreds of rows of many coefficients: the ratio for equally accurate kernels is 1 +- 0.1."""
    rc, plan = gpu.sig_plan(gpu.default_ctx(), B, L, d, 2, 1)
    assert rc == gpu.SIG_OK and plan.split_rows >= 1 and (plan.row_workgroups >= 1) == (d >= 10)
    x = workloads.brownian_paths(B, L, d, seed=9870 + d + L)
    mine, other = _errors(gpu, oracle, x, 2, [plan, copy_plan(plan, split_rows=0)], paths)
    assert mine <= 1.1 * other, (mine, other)


@pytest.mark.parametrize("d,B,L", [(2, 60003, 60), (5, 300, 70), (6, 4, 900), (10, 60, 200), (12, 40, 90), (20, 5, 700)])
def test_a_point_that_is_not_a_number_spoils_the_same_coefficients(gpu, d, B, L):  # noqa: F811
    """Behind a border of stretches and of workgroups too; sums that leave the range of a float likewise."""
    rc, plan = gpu.sig_plan(gpu.default_ctx(), B, L, d, 2, 1)
    assert rc == gpu.SIG_OK and plan.split_rows >= 1
    x = workloads.brownian_paths(B, L, d, seed=83)
    x[0, 5, 1] = np.nan
    x[1, (L - 1) // 2, d - 1] = np.nan
    x[B - 1, L - 1, 0] = np.nan
    x[2, 7:, :2] *= 1e25
    got = run_gpu(gpu, x, 2, True)
    plan.split_rows = 0
    other = run_gpu(gpu, x, 2, True, plan)
    assert np.array_equal(np.isnan(got[[0, 1, B - 1]]), np.isnan(other[[0, 1, B - 1]]))
    assert np.array_equal(np.isfinite(got[3:-1]), np.isfinite(other[3:-1])) and not np.isfinite(got[2, -1, d:]).all()
    assert np.isfinite(got[2, :, :d]).all() and not np.isfinite(got[2, -1, d]) and not np.isfinite(other[2, -1, d])


# whole paths, stretches of a path side by side (an infinite point at every border of them), and (few paths, several calls) at every
# border of workgroups
@pytest.mark.parametrize("d,B,L,segs", [(2, 60003, 60, 1), (3, 40001, 130, 1), (4, 6000, 60, 1), (5, 300, 70, 1), (8, 300, 150, 1), (9, 100, 80, 1), (4, 4, 900, 8),
                                        (6, 4, 900, 5), (10, 60, 200, 4), (12, 90, 90, 1), (20, 60, 60, 1), (13, 8000, 40, 1), (20, 5, 700, 16)])
def test_infinite_points(gpu, d, B, L, segs):  # noqa: F811
    rc, plan = gpu.sig_plan(gpu.default_ctx(), B, L, d, 2, 1)
    assert rc == gpu.SIG_OK
    sticky = d <= 10 and (plan.variant != gpu.SIG_VARIANT_LEVEL_SCAN or plan.row_workgroups > 0)
    slots, rows = 4 * (64 // d), -(-(L - 1) // segs)
    chunks = min(rows, slots)
    border = chunks * -(-rows // chunks)          # rows of a workgroup
    for first in ([0, 1, L - 1] + [w * border for w in range(1, segs) if w * border < L] if segs > 1 else [0]):
        x = infinite_points(B, L, d, 87 + d + first, first, 0 if segs > 1 else 1)
        plan.split_rows = segs
        got = run_gpu(gpu, x, 2, True, plan)
        plan.split_rows = 0
        assert_level1_is_added_up(x, got, run_gpu(gpu, x, 2, True, plan), sticky)
