"""Final-mode folds on matrix instructions (QuadTree in csrc/sig_onchip.h) against the fold of independent wavefronts, which does
the same multiply-adds one by one: the same bits.  Chunked plans and the fold with shared chains, which sum in another order,
against the fp64 oracle with the gates of test_gpu_parity.py."""
import numpy as np
import pytest

from paper_2501_08455_amd import workloads
from test_gpu_parity import check, gpu, run_gpu  # noqa: F401

pytestmark = pytest.mark.gpu

# d, depth, prefix depth: one and two levels below the lane's word; no, one, two and three letters outside the groups of four;
# lanes that fill up a path's last four ((9,3), (9,4), (11,3)) and paths of several workgroups with a ragged last one ((7,5), (9,4))
SHAPES = [(4, 3, 1), (4, 3, 2), (4, 4, 2), (4, 4, 3), (6, 3, 2), (6, 4, 2), (6, 4, 3), (8, 3, 2), (9, 3, 2), (9, 4, 2), (9, 4, 3), (10, 3, 2),
          (11, 3, 2), (7, 5, 3), (8, 4, 3), (4, 6, 4), (10, 4, 2)]


@pytest.mark.parametrize("d,depth,p", SHAPES)
def test_the_same_bits_as_vector_multiply_adds(gpu, d, depth, p):  # noqa: F811
    # (the last two: paths so small that whole levels are subnormal, which neither side may flush or round otherwise)
    small = 3e-13 if depth == 3 else 1e-10
    for B, L, scale in [(1, 2, 1.0), (3, 3, 1.0), (5, 20, 1.0), (300, 9, 1.0), (5, 20, small), (5, 20, small / 10)]:
        x = workloads.brownian_paths(B, L, d, seed=9500 + 31 * d + 7 * depth + L) * np.float32(scale)
        plans = [dict(), dict(tile_steps=2, tile_loader=2), dict(tile_steps=3, tile_loader=1), dict(threads=64), dict(threads=192)]
        want = run_gpu(gpu, x, depth, False, gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, prefix_depth=p, independent_waves=1))
        if scale != 1.0:
            assert np.count_nonzero((np.abs(want) < np.finfo(np.float32).tiny) & (want != 0)) > 20
        compared = 0
        for extra in plans:
            if extra.get("tile_steps", 0) > L - 1:
                continue
            plan = gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, prefix_depth=p, shared_chain=2, **extra)
            if gpu.sig_plan_validate(B, L, d, depth, 0, plan) != gpu.SIG_OK:
                continue
            assert np.array_equal(run_gpu(gpu, x, depth, False, plan), want), (B, L, extra)
            compared += 1
        assert compared >= (2 if L < 20 else 4), (B, L, compared)


@pytest.mark.parametrize("d,depth,p,chunks,segments", [(4, 3, 2, 16, 1), (4, 4, 2, 7, 2), (6, 3, 2, 7, 1), (8, 3, 2, 4, 3), (9, 3, 2, 3, 1),
                                                       (9, 3, 2, 2, 2), (11, 3, 2, 2, 1), (10, 3, 2, 2, 2), (8, 4, 2, 2, 1)])
def test_chunks_side_by_side(gpu, oracle, d, depth, p, chunks, segments):  # noqa: F811
    for B, L in [(1, 33), (5, 60), (2, 251)]:
        x = workloads.brownian_paths(B, L, d, seed=9600 + 31 * d + 7 * depth + L)
        check(gpu, oracle, x, depth, False, gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, prefix_depth=p, chunks=chunks, segments=segments), label="fours")


@pytest.mark.parametrize("d,depth,p", [(8, 4, 3), (9, 4, 3), (7, 5, 3), (5, 6, 4)])
def test_shared_chains(gpu, oracle, d, depth, p):  # noqa: F811
    for B, L in [(1, 2), (2, 4), (1, 60)]:
        x = workloads.brownian_paths(B, L, d, seed=9700 + 31 * d + 7 * depth + L)
        check(gpu, oracle, x, depth, False, gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, prefix_depth=p, shared_chain=1), label="shared")


def test_an_increment_that_is_not_finite_stays_in_its_path(gpu):  # noqa: F811
    for d, depth in [(9, 3), (4, 4), (8, 4)]:
        x = workloads.brownian_paths(7, 30, d, seed=9800 + d)
        clean = run_gpu(gpu, x, depth, False)
        x[3, 11, 2] = np.inf
        x[5, 0, d - 1] = np.nan
        got = run_gpu(gpu, x, depth, False)
        for b in range(7):
            if b not in (3, 5):
                assert np.array_equal(got[b], clean[b])
        assert not np.isfinite(got[3]).all() and np.isnan(got[5]).any()


@pytest.mark.parametrize("d,depth,p,B,L", [
    (4, 6, 4, 256, 50), (4, 6, 4, 257, 50), (4, 6, 4, 257, 40), (4, 6, 4, 6200, 5), (7, 5, 3, 128, 153), (7, 5, 3, 130, 153),
    (7, 5, 3, 130, 151), (7, 5, 3, 257, 153), (10, 5, 3, 896, 4), (10, 5, 3, 900, 4), (10, 5, 3, 900, 21), (6, 4, 3, 300, 20)])
def test_either_side_of_the_launches_that_keep_the_vector_fold(gpu, d, depth, p, B, L):  # noqa: F811
    x = workloads.brownian_paths(B, L, d, seed=9900 + d + B)
    want = run_gpu(gpu, x, depth, False, gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, prefix_depth=p, independent_waves=1))
    assert np.array_equal(run_gpu(gpu, x, depth, False, gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, prefix_depth=p, shared_chain=2)), want)
