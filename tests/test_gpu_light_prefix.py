"""Final mode at the borders of the planner's rule for light deeper entries (pick_on_chip in csrc/sig_api.hip): which prefix
depth is planned on either side, and the signature under that plan against the fp64 oracle with the gates of
test_gpu_parity.py.  Shapes whose lanes span workgroups have their border between two batches."""
import pytest

from paper_2501_08455_amd import workloads
from test_gpu_parity import check, gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,L,d,depth,p", [
    # nine and 48 increments, and one less and more
    (300, 9, 5, 4, 2), (300, 10, 5, 4, 3), (600, 49, 5, 4, 3), (600, 50, 5, 4, 2), (1500, 49, 7, 3, 2), (1500, 50, 7, 3, 1),
    (1200, 10, 5, 3, 2), (1200, 33, 6, 3, 2), (1300, 18, 3, 4, 2),
    # long paths only with two levels below the word: 500 increments and one less
    (1300, 500, 3, 4, 1), (1300, 501, 3, 4, 2), (1, 1200, 3, 4, 2), (3, 1200, 5, 3, 1), (3, 1200, 7, 3, 1),
    # the bound on the multiply-adds
    (4500, 10, 5, 4, 2), (3000, 1000, 3, 4, 1),
    # ... which is lower behind a lighter state
    (11000, 37, 5, 3, 2), (12000, 37, 5, 3, 1), (16000, 25, 5, 3, 2), (18500, 25, 5, 3, 1), (700, 48, 5, 4, 3), (860, 48, 5, 4, 2),
    # lanes in several workgroups: the last batch that takes them, and the next
    (320, 20, 8, 4, 3), (321, 20, 8, 4, 2), (252, 12, 9, 4, 3), (253, 12, 9, 4, 2), (204, 12, 10, 4, 3), (205, 12, 10, 4, 2),
    # ... and not where the shallower entry is cut in two segments, which sum half as many steps in a row
    (320, 96, 8, 4, 3), (256, 97, 8, 4, 2), (255, 97, 8, 4, 3), (252, 120, 9, 4, 3),
    # few lanes with states below 31 floats, and matrix instructions in place of the vector ones, as before
    (3000, 40, 3, 3, 1), (3000, 40, 4, 3, 1), (600, 30, 4, 4, 2)])
def test_prefix_depth_on_either_side_of_a_border(gpu, oracle, B, L, d, depth, p):  # noqa: F811
    rc, pl = gpu.sig_plan(None, B, L, d, depth, 0)
    assert rc == gpu.SIG_OK and pl.variant == gpu.SIG_VARIANT_ON_CHIP and pl.prefix_depth == p, pl.prefix_depth
    check(gpu, oracle, workloads.brownian_paths(B, L, d, seed=9900 + B + L), depth, False, pl, label="light")
