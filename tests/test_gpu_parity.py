"""GPU parity: libsig (through the C ABI binding) against the fp64 oracle, element by element.

Gates, per level n of the output rows (Eq. 10), all at the stated tolerance 1e-4:
  aggregate  ||gpu_n - oracle_n||_F / ||oracle_n||_F over every emitted row of the call (the stated metric);
  per row    the same ratio for every single row (B rows, or B x (L-1) in stream mode), so that one wrong or
             stale row cannot hide among thousands of right ones; rows whose oracle norm is below 1e-30
             (repeated points: an exactly zero signature) are compared absolutely;
  element    |gpu - oracle| <= 1e-4 x max|oracle_n| over the call, for every coefficient.
Rows of a path that has come back towards its start have a small level-n norm that still carries the rounding
error of the earlier, larger prefixes; the per-row figure therefore divides by max(||oracle row||, r^n / n!) with r
the largest distance of the row's prefix from its first point (what level n reaches along a straight path of that
extent; computed from the input alone, and small for the early rows of a stream, which stay strictly gated).
The aggregate over these row scales is also held to a bound derived from the arithmetic (fp32 unit roundoff
u = 2^-24, K increments folded one after the other: 20 u sqrt(K), at most 1e-4); measured: at most 2.8 u sqrt(K).
Outputs are poisoned with NaN before the call, so a coefficient the kernels never write fails the finiteness check.
"""
import sys

import numpy as np
import pytest

from paper_2501_08455_amd import workloads

pytestmark = pytest.mark.gpu

TOL = 1e-4
UNIT_ROUNDOFF = 2.0 ** -24


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2501_08455_amd import binding
    binding.load()
    return binding


def say(msg):
    print(msg)
    sys.stdout.flush()


def level_errors(got, want, d, depth):
    got = np.asarray(got, dtype=np.float64).reshape(-1, got.shape[-1])
    want = want.reshape(-1, want.shape[-1])
    errs, start = [], 0
    for n in range(1, depth + 1):
        sl = slice(start, start + d ** n)
        num = np.linalg.norm(got[:, sl] - want[:, sl])
        den = np.linalg.norm(want[:, sl])
        errs.append(num / den if den > 0 else num)
        start += d ** n
    return errs


def row_scales(x, depth, stream):
    """Per emitted row and level n: r^n / n! with r the largest distance of the row's prefix of the path from its
    first point, the size level n reaches somewhere along a straight path of that extent.  A row whose level-n
    norm lies far below this has come back towards its start; the rounding error of its earlier, larger prefixes
    remains in it, so its error is measured against this scale rather than against its own small norm."""
    x = np.asarray(x, dtype=np.float64)
    r = np.maximum.accumulate(np.linalg.norm(x[:, 1:] - x[:, :1], axis=2), axis=1)   # [B][K]
    r = r if stream else r[:, -1:]
    fact = np.cumprod(np.arange(1, depth + 1, dtype=np.float64))
    return np.stack([r.reshape(-1) ** n / fact[n - 1] for n in range(1, depth + 1)], axis=1)   # [rows][depth]


def row_and_element_errors(got, want, d, depth, scales):
    """Per level: (worst per-row relative error, its row, worst |difference| over max|oracle| of the level,
    aggregate error over the rows' norms or scales, whichever is larger)."""
    got = np.asarray(got, dtype=np.float64).reshape(-1, got.shape[-1])
    want = want.reshape(-1, want.shape[-1])
    res, start = [], 0
    for n in range(1, depth + 1):
        sl = slice(start, start + d ** n)
        diff = got[:, sl] - want[:, sl]
        num = np.sqrt(np.einsum("ij,ij->i", diff, diff))
        den = np.maximum(np.sqrt(np.einsum("ij,ij->i", want[:, sl], want[:, sl])), scales[:, n - 1])
        rel = np.where(den > 1e-30, num / np.maximum(den, 1e-30), num)
        worst = int(np.argmax(rel))
        top = float(np.max(np.abs(want[:, sl])))
        elem = float(np.max(np.abs(diff))) / top if top > 0 else float(np.max(np.abs(diff)))
        agg = float(np.linalg.norm(num)) / max(float(np.linalg.norm(den)), 1e-30)
        res.append((float(rel[worst]), worst, elem, agg))
        start += d ** n
    return res


def aggregate_bound(K):
    """What fp32 arithmetic allows the aggregate figure: 20 u sqrt(K) for K increments, never above the stated 1e-4."""
    return min(TOL, 20.0 * UNIT_ROUNDOFF * np.sqrt(max(K, 1)))


def assert_parity(got, want, x, depth, stream, arithmetic_bound=True):
    """The gates of the module docstring; `x` is the batch of paths the rows of `got` and `want` belong to.
    arithmetic_bound=False leaves out the bound derived from the arithmetic (the level-by-level family on one
    channel: its sums over time add terms of both signs that are larger than their total)."""
    d, K = x.shape[2], x.shape[1] - 1
    assert got.shape == want.shape
    assert np.all(np.isfinite(got))
    errs = level_errors(got, want, d, depth)
    rows = row_and_element_errors(got, want, d, depth, row_scales(x, depth, stream))
    say("  per-level rel err: " + " ".join("%.2e" % e for e in errs))
    say("  worst row (rel err @ row): " + " ".join("%.2e@%d" % (r[0], r[1]) for r in rows) +
        " | worst element / max: " + " ".join("%.2e" % r[2] for r in rows) +
        " | aggregate over row scales: " + " ".join("%.2e" % r[3] for r in rows) + " bound %.2e" % aggregate_bound(K))
    assert max(errs) <= TOL, errs
    assert max(r[0] for r in rows) <= TOL, rows
    assert max(r[2] for r in rows) <= TOL, rows
    assert not arithmetic_bound or max(r[3] for r in rows) <= aggregate_bound(K), (rows, aggregate_bound(K))


def run_gpu(gpu, x, depth, stream, plan=None):
    import torch
    xt = torch.from_numpy(x).cuda()
    B, L, d = x.shape
    D = gpu.sig_size(d, depth)
    out = torch.full((B, L - 1, D) if stream else (B, D), float("nan"), dtype=torch.float32, device="cuda")
    out = gpu.signature(xt, depth, stream=stream, plan=plan, out=out)
    torch.cuda.synchronize()
    return out.cpu().numpy()


def check(gpu, oracle, x, depth, stream, plan=None, label="", arithmetic_bound=True):
    say("case %s shape=%s depth=%d stream=%s plan=%s" % (label, x.shape, depth, stream,
                                                        plan.as_dict() if plan is not None else "auto"))
    got = run_gpu(gpu, x, depth, stream, plan)
    want = oracle.signature(x, depth, stream=stream)
    assert_parity(got, want, x, depth, stream, arithmetic_bound)
    return got


# ---------------------------------------------------------------- the five configurations, automatic plan
@pytest.mark.parametrize("name", ["C1", "C2", "C3", "C4", "C5"])
def test_config_auto_plan(gpu, oracle, name):
    cfg = workloads.CONFIGS[name]
    x = workloads.make_paths(cfg)
    check(gpu, oracle, x, cfg.depth, cfg.stream, label=name)


# ---------------------------------------------------------------- HBM-streaming family on shapes with and without compiled kernels
@pytest.mark.parametrize("B,L,d,depth,stream,p", [
    (4, 16, 2, 3, False, 0), (4, 16, 2, 3, True, 1), (3, 9, 3, 5, False, 2), (3, 9, 3, 5, True, 0),
    (2, 40, 5, 4, False, 1), (2, 40, 5, 4, True, 3), (5, 7, 1, 6, False, 0), (5, 7, 1, 6, True, 0),
    (2, 12, 7, 2, False, 1), (2, 12, 6, 1, True, 0), (1, 130, 2, 10, False, 3), (2, 70, 4, 4, True, 2),
    (1, 20, 10, 5, False, 2), (3, 2, 3, 4, False, 0), (3, 2, 3, 4, True, 1),
])
def test_hbm_streaming_family(gpu, oracle, B, L, d, depth, stream, p):
    rng = np.random.default_rng(1000 + B + L + d + depth)
    x = np.cumsum(rng.normal(0, 0.3, size=(B, L, d)), axis=1).astype(np.float32)
    plan = gpu.make_plan(gpu.SIG_VARIANT_HBM_STREAMING, prefix_depth=p)
    check(gpu, oracle, x, depth, stream, plan, label="hbm")


def test_uncompiled_shapes_fall_back(gpu, oracle):
    for (B, L, d, depth) in [(3, 33, 7, 6), (2, 17, 1, 4), (130, 5, 3, 7), (3, 20, 12, 3), (2, 40, 2, 9), (5, 9, 16, 2)]:
        rc, pl = gpu.sig_plan(None, B, L, d, depth, 0)
        fits_level_scan = d <= 256 and depth <= 8
        assert rc == 0 and pl.variant == (gpu.SIG_VARIANT_LEVEL_SCAN if fits_level_scan else gpu.SIG_VARIANT_HBM_STREAMING)
        x = workloads.brownian_paths(B, L, d, seed=77 + d)
        check(gpu, oracle, x, depth, False, label="fallback")
        check(gpu, oracle, x, depth, True, label="fallback-stream")


# ---------------------------------------------------------------- on-chip family: every compiled kernel, several time cuttings
ON_CHIP_CASES = [
    # d, depth, p, B, L, chunks, segments, tile_steps, stream[, threads]
    (2, 3, 0, 300, 16, 1, 1, 0, False), (2, 3, 0, 7, 41, 4, 2, 3, False), (2, 3, 0, 5, 41, 5, 1, 0, True),
    (2, 3, 1, 4, 16, 1, 1, 0, False), (2, 3, 1, 4, 16, 1, 1, 0, True), (2, 3, 1, 9, 100, 7, 3, 4, False),
    (2, 3, 1, 3, 100, 9, 1, 5, True),
    (4, 4, 1, 70, 37, 1, 1, 0, False), (4, 4, 1, 70, 37, 1, 1, 5, True, 64), (4, 4, 1, 3, 256, 8, 4, 0, False),
    (4, 4, 1, 5, 256, 16, 1, 0, True), (4, 4, 2, 64, 256, 16, 1, 0, True), (4, 4, 2, 3, 100, 3, 5, 7, False),
    (4, 4, 2, 20, 50, 1, 1, 0, True),
    (5, 4, 1, 128, 100, 1, 1, 0, False), (5, 4, 1, 60, 23, 1, 1, 3, True, 64), (5, 4, 1, 2, 333, 10, 4, 0, False),
    (5, 4, 1, 3, 90, 6, 1, 0, True),
    (5, 4, 2, 128, 100, 10, 1, 0, False), (5, 4, 2, 128, 100, 5, 2, 4, False), (5, 4, 2, 11, 100, 1, 1, 0, False),
    (5, 4, 2, 2, 2000, 10, 8, 0, False), (5, 4, 2, 3, 700, 3, 13, 9, False), (5, 4, 2, 4, 61, 4, 1, 0, True), (5, 4, 2, 13, 30, 1, 1, 0, True),
    (10, 6, 4, 2, 9, 1, 1, 0, False), (10, 6, 4, 1, 4, 1, 1, 2, True),
    (5, 4, 2, 40, 100, 7, 1, 0, False, 512), (4, 4, 2, 9, 256, 16, 1, 0, True, 512), (5, 4, 2, 9000, 30, 1, 1, 7, False),
    (4, 4, 2, 3000, 20, 1, 1, 6, True), (2, 3, 1, 70000, 9, 1, 1, 0, False), (5, 4, 2, 33, 300, 1, 4, 0, False, 128),
    # the deeper prefix of five channels at depth 4 (125 lanes per path): the plan of small batches of short paths
    # (four chunks in 512 threads), two chunks in 256, uncut, cut into segments, tiled, and in stream mode
    (5, 4, 3, 128, 100, 4, 1, 0, False, 512), (5, 4, 3, 7, 33, 2, 1, 0, False), (5, 4, 3, 3, 20, 1, 1, 0, False),
    (5, 4, 3, 5, 257, 4, 3, 0, False, 512), (5, 4, 3, 300, 64, 3, 1, 5, False, 512), (5, 4, 3, 6, 41, 2, 1, 0, True),
    (5, 4, 3, 2, 2, 1, 1, 0, False),
    # workgroups of 512 threads for the other small lane states with more than 64 lanes per path
    (5, 5, 3, 9, 100, 4, 1, 0, False, 512), (5, 5, 3, 3, 500, 4, 2, 0, False, 512), (6, 5, 3, 5, 77, 2, 1, 0, False, 512),
    (6, 5, 3, 2, 400, 2, 4, 0, False, 512), (9, 3, 2, 20, 100, 6, 1, 0, False, 512), (9, 3, 2, 3, 1000, 6, 6, 0, False, 512),
    (10, 3, 2, 11, 130, 5, 2, 0, False, 512), (10, 3, 2, 300, 60, 4, 1, 7, False, 512),
    # the deeper prefix of (4,4), (5,3) and (6,3): the planner's small-batch plans, cut and tiled ones, and stream mode
    (4, 4, 3, 128, 100, 8, 1, 0, False, 512), (4, 4, 3, 5, 50, 4, 1, 0, False), (4, 4, 3, 3, 300, 8, 2, 0, False, 512),
    (4, 4, 3, 70, 64, 2, 1, 5, False), (4, 4, 3, 6, 41, 2, 1, 0, True), (4, 4, 3, 2, 9, 1, 1, 0, True),
    (5, 3, 2, 128, 100, 8, 1, 0, False), (5, 3, 2, 9, 257, 16, 1, 0, False, 512), (5, 3, 2, 4, 500, 10, 3, 0, False),
    (5, 3, 2, 300, 40, 3, 1, 6, False), (5, 3, 2, 7, 33, 4, 1, 0, True), (5, 3, 2, 2, 2, 1, 1, 0, False),
    (6, 3, 2, 128, 100, 7, 1, 0, False), (6, 3, 2, 11, 200, 14, 1, 0, False, 512), (6, 3, 2, 3, 400, 7, 4, 0, False),
    (6, 3, 2, 200, 30, 2, 1, 4, False), (6, 3, 2, 5, 29, 3, 1, 0, True),
    # ... and of (4,3), (7,3), (3,4), (3,5), (2,6), (3,6)
    (4, 3, 2, 128, 100, 12, 1, 0, False), (4, 3, 2, 9, 257, 32, 1, 0, False, 512), (4, 3, 2, 5, 300, 8, 3, 0, False), (4, 3, 2, 7, 33, 4, 1, 0, True),
    (7, 3, 2, 128, 100, 8, 1, 0, False, 512), (7, 3, 2, 64, 20, 1, 1, 0, False), (7, 3, 2, 3, 400, 5, 4, 0, False), (7, 3, 2, 6, 25, 2, 1, 0, True),
    (3, 4, 2, 128, 100, 12, 1, 0, False), (3, 4, 2, 11, 257, 28, 1, 0, False), (3, 4, 2, 300, 40, 3, 1, 6, False), (3, 4, 2, 5, 31, 4, 1, 0, True),
    (3, 5, 3, 128, 100, 8, 1, 0, False), (3, 5, 3, 9, 200, 16, 1, 0, False, 512), (3, 5, 3, 2, 500, 8, 4, 0, False), (3, 5, 3, 4, 27, 2, 1, 0, True),
    (2, 6, 2, 128, 100, 12, 1, 0, False), (2, 6, 2, 7, 257, 32, 1, 0, False), (2, 6, 2, 3, 600, 16, 3, 0, False), (2, 6, 2, 5, 40, 4, 1, 0, True),
    (3, 6, 4, 128, 100, 6, 1, 0, False, 512), (3, 6, 4, 64, 20, 2, 1, 0, False, 512), (3, 6, 4, 2, 300, 3, 4, 0, False), (3, 6, 4, 3, 19, 2, 1, 0, True),
    # ... and (3,3), (2,4), (3,4) one deeper, (2,5), (2,6) one deeper, (6,4)
    (3, 3, 2, 128, 100, 12, 1, 0, False), (3, 3, 2, 9, 257, 28, 1, 0, False), (3, 3, 2, 5, 300, 8, 3, 0, False), (3, 3, 2, 7, 33, 4, 1, 0, True),
    (2, 4, 2, 128, 100, 12, 1, 0, False), (2, 4, 2, 9, 257, 32, 1, 0, False), (2, 4, 2, 5, 300, 8, 3, 0, False), (2, 4, 2, 7, 33, 4, 1, 0, True),
    (3, 4, 3, 128, 100, 8, 1, 0, False), (3, 4, 3, 9, 257, 16, 1, 0, False, 512), (3, 4, 3, 5, 300, 8, 3, 0, False), (3, 4, 3, 7, 33, 4, 1, 0, True),
    (2, 5, 2, 128, 100, 12, 1, 0, False), (2, 5, 2, 9, 257, 32, 1, 0, False), (2, 5, 2, 300, 40, 3, 1, 6, False), (2, 5, 2, 7, 33, 4, 1, 0, True),
    (2, 6, 3, 128, 100, 8, 1, 0, False), (2, 6, 3, 9, 257, 32, 1, 0, False), (2, 6, 3, 5, 300, 8, 3, 0, False), (2, 6, 3, 7, 33, 4, 1, 0, True),
    (6, 4, 3, 128, 100, 2, 1, 0, False, 512), (6, 4, 3, 64, 20, 1, 1, 0, False), (6, 4, 3, 3, 300, 2, 4, 0, False, 512), (6, 4, 3, 4, 21, 1, 1, 0, True),
    (6, 4, 3, 50, 64, 1, 1, 5, False),
]


# time segments whose partial rows are too long for the LDS of a join kernel: joined in device memory by a pairwise tree
# of batched row products (a power of two of segments, up to 32); lane states above 64 floats, lanes of a path
# within one workgroup ((10,4), (8,4), (6,5)) and across several ((7,5): 343 lanes), ragged and empty last segments
TREE_JOIN_CASES = [
    # d, depth, p, B, L, segments, tile_steps
    (10, 4, 2, 1, 700, 8, 0), (10, 4, 2, 3, 333, 4, 0), (10, 4, 2, 2, 65, 32, 0), (8, 4, 2, 5, 200, 16, 7),
    (6, 5, 3, 2, 150, 8, 0), (7, 5, 3, 1, 130, 4, 0), (7, 5, 3, 2, 97, 16, 0), (9, 4, 2, 1, 40, 32, 0),
    (4, 6, 4, 1, 90, 8, 0),
    # the deeper prefix of 8 and 10 channels at depth 4 (512 / 1,000 lanes per path), uncut and cut
    (10, 4, 3, 3, 50, 1, 0), (8, 4, 3, 2, 300, 8, 0), (8, 4, 3, 3, 60, 2, 0), (9, 4, 3, 2, 41, 2, 0), (10, 4, 3, 1, 600, 16, 0), (8, 4, 3, 40, 23, 1, 5),
    (9, 4, 3, 5, 77, 1, 0), (9, 4, 3, 1, 400, 4, 0),
]


@pytest.mark.parametrize("case", TREE_JOIN_CASES, ids=lambda c: "-".join(str(v) for v in c))
def test_on_chip_segments_joined_in_device_memory(gpu, oracle, case):
    d, depth, p, B, L, segments, tile = case
    assert gpu.sig_on_chip_available(d, depth, p)
    x = workloads.brownian_paths(B, L, d, seed=5200 + 17 * B + L + segments)
    plan = gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, prefix_depth=p, chunks=1, segments=segments, tile_steps=tile)
    check(gpu, oracle, x, depth, False, plan, label="on-chip, tree join")
    # not a power of two, or more than 32: refused on the host
    for bad in (3, 6, 64):
        if segments > 1 and bad * gpu.sig_size(d, depth) * 4 > 64 * 1024:
            bad_plan = gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, prefix_depth=p, chunks=1, segments=bad)
            assert gpu.sig_plan_validate(B, L, d, depth, 0, bad_plan) == gpu.SIG_ERR_INVALID


@pytest.mark.parametrize("d,depth,B,L", [(10, 4, 1, 1000), (8, 4, 3, 2000), (7, 5, 1, 600), (6, 5, 2, 900), (4, 6, 1, 1500)])
def test_few_long_paths_with_large_states_auto(gpu, oracle, d, depth, B, L):
    """The planner cuts few long paths of shapes with large lane states into tree-joined segments."""
    rc, pl = gpu.sig_plan(gpu.default_ctx(), B, L, d, depth, 0)
    assert rc == gpu.SIG_OK and pl.variant == gpu.SIG_VARIANT_ON_CHIP and pl.segments >= 4
    x = workloads.brownian_paths(B, L, d, seed=5300 + L)
    check(gpu, oracle, x, depth, False, None, label="auto, tree join")


# Shapes whose lanes per path exceed a workgroup, final mode: the fold that reads the shared prefix part of the Horner
# chains from a table in LDS (shared_chain = 1; the whole (path, segment) is one tile, so it takes segments of up to
# 16 steps per table-building thread: 128 for ten channels, fewer for five) and, with shared_chain = 2, the fold in which
# every lane carries its own prefix chain.  Time segments (ragged and empty last ones), workgroups of 64 to 256 threads
# (the last workgroup of a path is partly idle: 10^4 = 39 x 256 + 16), one-step paths.
SHARED_CHAIN_CASES = [
    # d, depth, p, B, L, segments, threads
    (10, 6, 4, 2, 30, 1, 256), (10, 6, 4, 1, 128, 1, 256), (10, 6, 4, 1, 23, 2, 128), (10, 6, 4, 1, 9, 1, 64),
    (10, 6, 4, 1, 300, 4, 256), (8, 4, 3, 3, 60, 1, 256), (8, 4, 3, 2, 300, 8, 256), (10, 4, 3, 5, 128, 1, 256),
    (10, 4, 3, 1, 1000, 8, 128), (9, 4, 3, 2, 33, 1, 64), (7, 5, 3, 2, 60, 1, 256), (7, 5, 3, 1, 200, 4, 256),
    (10, 5, 3, 1, 50, 1, 256), (8, 5, 3, 1, 45, 2, 256), (9, 5, 3, 1, 31, 1, 128), (5, 6, 4, 3, 60, 1, 256),
    (5, 6, 4, 1, 400, 8, 256), (10, 4, 3, 3, 2, 1, 256), (8, 4, 3, 40, 23, 1, 256),
]


@pytest.mark.parametrize("case", SHARED_CHAIN_CASES, ids=lambda c: "-".join(str(v) for v in c))
def test_shared_prefix_chain_fold(gpu, oracle, case):
    d, depth, p, B, L, segments, threads = case
    assert gpu.sig_on_chip_available(d, depth, p)
    x = workloads.brownian_paths(B, L, d, seed=5600 + 17 * B + L + segments)
    outs = []
    for mode in (1, 2):
        plan = gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, prefix_depth=p, chunks=1, segments=segments, threads=threads,
                             shared_chain=mode)
        assert gpu.sig_plan_validate(B, L, d, depth, 0, plan) == gpu.SIG_OK, (mode, case)
        outs.append(check(gpu, oracle, x, depth, False, plan, label="shared chain %d" % mode))
    # different evaluation orders of the same sums: equal to rounding
    assert max(level_errors(outs[0], outs[1].astype(np.float64), d, depth)) <= 1e-6


def test_shared_prefix_chain_fold_is_refused_where_it_does_not_fit(gpu):
    """One tile per (path, segment): segments longer than the table builders can take, forced tiles and stream mode have
    no such kernel; neither have shapes whose lanes fit a workgroup."""
    for (B, L, d, depth, p, kw) in [(1, 300, 10, 6, 4, {}), (1, 100, 10, 6, 4, {"tile_steps": 7}), (1, 100, 5, 6, 4, {}),
                                    (2, 50, 5, 4, 2, {}), (2, 50, 6, 4, 3, {})]:
        plan = gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, prefix_depth=p, shared_chain=1, **kw)
        assert gpu.sig_plan_validate(B, L, d, depth, 0, plan) == gpu.SIG_ERR_INVALID, (B, L, d, depth, p, kw)
    plan = gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, prefix_depth=4, shared_chain=1)
    assert gpu.sig_plan_validate(1, 100, 10, 6, 1, plan) == gpu.SIG_ERR_INVALID
    assert gpu.sig_plan_validate(1, 100, 10, 6, 0, plan) == gpu.SIG_OK


def split_case(case):
    d, depth, p, B, L, chunks, segments, tile, stream = case[:9]
    threads = case[9] if len(case) > 9 else 256
    return d, depth, p, B, L, chunks, segments, tile, stream, threads


@pytest.mark.parametrize("case", ON_CHIP_CASES, ids=lambda c: "-".join(str(v) for v in c))
def test_on_chip_family(gpu, oracle, case):
    d, depth, p, B, L, chunks, segments, tile, stream, threads = split_case(case)
    assert gpu.sig_on_chip_available(d, depth, p)
    x = workloads.brownian_paths(B, L, d, seed=5000 + 17 * B + L + chunks)
    plan = gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, prefix_depth=p, chunks=chunks, segments=segments,
                         tile_steps=tile, threads=threads)
    check(gpu, oracle, x, depth, stream, plan, label="on-chip")


@pytest.mark.parametrize("loader", [1, 2], ids=["staged", "plain"])
@pytest.mark.parametrize("case", [c for c in ON_CHIP_CASES if c[7] > 0], ids=lambda c: "-".join(str(v) for v in c))
def test_on_chip_tile_loaders(gpu, oracle, case, loader):
    """Plans with several tiles per chunk, with either loader (plan.tile_loader) forced."""
    d, depth, p, B, L, chunks, segments, tile, stream, threads = split_case(case)
    x = workloads.brownian_paths(B, L, d, seed=9000 + 11 * B + L + loader)
    plan = gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, prefix_depth=p, chunks=chunks, segments=segments,
                         tile_steps=tile, threads=threads, tile_loader=loader)
    if gpu.sig_plan_validate(B, L, d, depth, int(stream), plan) != gpu.SIG_OK:
        pytest.skip("plan not valid with this loader")
    check(gpu, oracle, x, depth, stream, plan, label="tile loader %d" % loader)


@pytest.mark.parametrize("case", [c for c in ON_CHIP_CASES if c[5] == 1], ids=lambda c: "-".join(str(v) for v in c))
def test_on_chip_independent_wavefronts(gpu, oracle, case):
    """The barrier-free variant of the single-chunk kernels (plan.independent_waves = 1)."""
    d, depth, p, B, L, chunks, segments, tile, stream, threads = split_case(case)
    x = workloads.brownian_paths(B, L, d, seed=7000 + 13 * B + L)
    plan = gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, prefix_depth=p, chunks=1, segments=segments,
                         tile_steps=tile, threads=threads, independent_waves=1)
    if gpu.sig_plan_validate(B, L, d, depth, int(stream), plan) != gpu.SIG_OK:
        pytest.skip("plan not valid for this variant")
    check(gpu, oracle, x, depth, stream, plan, label="independent")


# ---------------------------------------------------------------- the wider shape grid (channels 2..10, depths 2..6)
SHAPE_GRID = [(2, 2, 1), (3, 2, 1), (4, 2, 1), (5, 2, 1), (6, 2, 1), (8, 2, 1), (10, 2, 1),
              (3, 3, 1), (4, 3, 1), (5, 3, 1), (6, 3, 1), (7, 3, 1), (8, 3, 2), (10, 3, 2),
              (2, 4, 1), (3, 4, 1), (6, 4, 2), (7, 4, 2), (8, 4, 2), (10, 4, 2),
              (2, 5, 1), (3, 5, 2), (4, 5, 3), (5, 5, 3), (6, 5, 3), (2, 6, 1), (3, 6, 3), (4, 6, 4), (5, 6, 4),
              (7, 2, 1), (9, 2, 1), (9, 3, 2), (9, 4, 2), (7, 5, 3), (8, 5, 3), (9, 5, 3), (10, 5, 3)]


@pytest.mark.parametrize("shape", SHAPE_GRID, ids=lambda c: "-".join(str(v) for v in c))
def test_shape_grid(gpu, oracle, shape):
    """Every further compiled kernel: the planner's choice at two batch sizes, and forced time cuts."""
    d, depth, p = shape
    assert gpu.sig_on_chip_available(d, depth, p)
    Q = d ** p
    for B, L in [(3, 23), (70, 9)]:
        x = workloads.brownian_paths(B, L, d, seed=6000 + 31 * d + depth + B)
        for stream in (False, True):
            rc, pl = gpu.sig_plan(None, B, L, d, depth, int(stream))
            assert rc == gpu.SIG_OK
            # (stream mode with few paths may take the level-by-level family; the forced plans below and
            # test_on_chip_cases cover the register kernels' stream paths)
            assert pl.variant in (gpu.SIG_VARIANT_ON_CHIP, gpu.SIG_VARIANT_LEVEL_SCAN)
            check(gpu, oracle, x, depth, stream, label="grid auto")
            if stream and pl.row_workgroups > 0:
                pl.row_workgroups = 0
                check(gpu, oracle, x, depth, stream, pl, label="grid, without rows from registers")
    x = workloads.brownian_paths(4, 41, d, seed=6100 + d + depth)
    forced = [(1, 3, 4, False), (1, 1, 7, True)]
    if Q <= 64:
        forced += [(3, 2, 0, False), (2, 1, 0, True), (3, 1, 5, True)]
    ran = 0
    for chunks, segments, tile, stream in forced:
        for threads in (256, 128, 64):
            plan = gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, prefix_depth=p, chunks=chunks, segments=segments,
                                 tile_steps=tile, threads=threads)
            if gpu.sig_plan_validate(4, 41, d, depth, int(stream), plan) == gpu.SIG_OK:
                check(gpu, oracle, x, depth, stream, plan, label="grid forced")
                ran += 1
                break
        else:
            # long rows: the rows of all chunks / segments of a path do not fit LDS at any workgroup size
            say("plan %r does not fit this shape" % ((chunks, segments, tile, stream),))
    assert ran >= 1


def test_single_increment_and_repeated_points(gpu, oracle):
    x = workloads.brownian_paths(6, 2, 5, seed=3)
    check(gpu, oracle, x, 4, False, label="L=2")
    check(gpu, oracle, x, 4, True, label="L=2 stream")
    y = workloads.brownian_paths(3, 20, 4, seed=4)
    y[:, 5] = y[:, 4]
    y[:, 11:14] = y[:, 10:11]
    check(gpu, oracle, y, 4, True, label="repeated points")


def test_error_codes_and_empty_batch(gpu):
    import torch
    ctx = gpu.default_ctx()
    x = torch.zeros((2, 5, 3), device="cuda")
    out = torch.zeros((2, gpu.sig_size(3, 2)), device="cuda")
    assert gpu.sig_compute(ctx, x, 2, 0, out) == gpu.SIG_OK
    assert gpu.sig_compute(ctx, x, 0, 0, out) == gpu.SIG_ERR_INVALID
    assert gpu.sig_compute(ctx, x, 2, 2, out) == gpu.SIG_ERR_INVALID
    assert gpu.sig_compute(ctx, x[:, :1].contiguous(), 2, 0, out) == gpu.SIG_ERR_INVALID
    assert gpu.sig_compute(ctx, x, 40, 0, out) == gpu.SIG_ERR_TOO_LARGE
    assert gpu.sig_compute(None, x, 2, 0, out) == gpu.SIG_ERR_INVALID
    empty = torch.zeros((0, 5, 3), device="cuda")
    assert gpu.sig_compute(ctx, empty, 2, 0, out) == gpu.SIG_OK
    bad = gpu.make_plan(gpu.SIG_VARIANT_ON_CHIP, prefix_depth=0, chunks=1, segments=1)
    assert gpu.sig_compute(ctx, x, 2, 0, out, plan=bad) == gpu.SIG_ERR_INVALID  # (3, 2) has no kernel with p = 0
    torch.cuda.synchronize()


def test_runs_are_bitwise_reproducible(gpu):
    for name in ["C2", "C4"]:
        cfg = workloads.CONFIGS[name]
        x = workloads.make_paths(cfg)
        a = run_gpu(gpu, x, cfg.depth, cfg.stream)
        b = run_gpu(gpu, x, cfg.depth, cfg.stream)
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("d,depth,B", [(3, 4, 37), (5, 4, 300), (1, 6, 5), (2, 1, 9), (10, 6, 2), (7, 3, 70000), (13, 2, 11),
                                        (2, 25, 1),
                                        # batches of short rows, several rows to a workgroup: a ragged last workgroup,
                                        # one to ten rows per workgroup, the longest rows that kernel takes
                                        (5, 4, 2049), (4, 4, 4100), (2, 6, 3001), (6, 4, 2500), (3, 7, 2100), (8, 2, 9000),
                                        (2, 3, 5000), (2, 2, 3000), (3, 2, 2500)])
def test_sig_combine_matches_eq4(gpu, oracle, d, depth, B):
    """Batched truncated product (Eq. 4) against the oracle's; (2, 25) has levels of more than 2^24 words, where the
    kernel's index arithmetic takes its integer-division path."""
    import torch
    D = gpu.sig_size(d, depth)
    rng = np.random.default_rng(9)
    a = (rng.normal(size=(B, D)) * 0.5).astype(np.float32)
    b = (rng.normal(size=(B, D)) * 0.5).astype(np.float32)
    out = torch.full((B, D), float("nan"), device="cuda")
    rc = gpu.sig_combine(gpu.default_ctx(), torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda(), d, depth, out)
    assert rc == gpu.SIG_OK
    torch.cuda.synchronize()
    pick = np.arange(B) if B <= 300 else np.random.default_rng(1).choice(B, size=64, replace=False)
    want = np.stack([oracle.tensor_mul(np.concatenate([[1.0], a[i]]), np.concatenate([[1.0], b[i]]), d, depth)[1:]
                     for i in pick])
    got = out.cpu().numpy()[pick]
    assert np.all(np.isfinite(got))
    assert max(level_errors(got, want, d, depth)) <= 1e-5


# ---------------------------------------------------------------- batch-saturated variants, checked on a sample of paths
@pytest.mark.parametrize("name,B", [("C2", 65536), ("C3", 4096), ("C4", 4096), ("C1", 1 << 20)])
def test_saturated_variants_sampled(gpu, oracle, name, B):
    import torch
    cfg = workloads.CONFIGS[name]
    x = workloads.make_paths(cfg, B=B, seed=99)
    say("case %s-sat B=%d" % (name, B))
    xt = torch.from_numpy(x).cuda()
    D = gpu.sig_size(cfg.d, cfg.depth)
    out = torch.full((B, cfg.L - 1, D) if cfg.stream else (B, D), float("nan"), dtype=torch.float32, device="cuda")
    gpu.signature(xt, cfg.depth, stream=cfg.stream, out=out)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(out).all())      # every row of the whole batch was written
    rng = np.random.default_rng(5)
    pick = np.sort(rng.choice(B, size=128, replace=False))
    pick[0], pick[-1] = 0, B - 1
    got = out[torch.from_numpy(pick).cuda()].cpu().numpy()
    want = oracle.signature(x[pick], cfg.depth, stream=cfg.stream)
    assert_parity(got, want, x[pick], cfg.depth, cfg.stream)


# ---------------------------------------------------------------- long paths and very large batches
@pytest.mark.parametrize("B,L,d,depth,stream", [(3, 50000, 5, 4, False), (2, 20000, 4, 4, True),
                                                (1, 100000, 2, 3, False), (5, 3000, 10, 3, False)])
def test_long_paths(gpu, oracle, B, L, d, depth, stream):
    x = workloads.brownian_paths(B, L, d, seed=300 + L)
    check(gpu, oracle, x, depth, stream, label="long path")


def test_very_large_batch_sampled(gpu, oracle):
    import torch
    B, L, d, depth = 1 << 21, 3, 2, 3
    x = workloads.brownian_paths(B, L, d, seed=17)
    out = torch.full((B, gpu.sig_size(d, depth)), float("nan"), dtype=torch.float32, device="cuda")
    gpu.signature(torch.from_numpy(x).cuda(), depth, out=out)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(out).all())
    pick = np.concatenate([np.array([0, 1, 255, 256, 65535, 65536, B // 2, B - 2, B - 1]),
                           np.random.default_rng(6).choice(B, size=247, replace=False)])
    got = out[torch.from_numpy(pick).cuda()].cpu().numpy()
    want = oracle.signature(x[pick], depth)
    assert_parity(got, want, x[pick], depth, False)


def test_path_array_of_more_than_2_31_floats(gpu, oracle):
    """A batch whose path array holds 2.5e9 floats (10 GB): offsets into it do not fit 32 bits.  The straight-copy tile
    loader of the first workgroups, the one of the last (which clamps its reads to the end of the array) and paths in
    between are checked against the oracle; every output row must have been written."""
    import torch
    B, L, d, depth = 5_000_000, 100, 5, 4
    rc, pl = gpu.sig_plan(gpu.default_ctx(), B, L, d, depth, 0)
    assert rc == gpu.SIG_OK
    say("case 2^31 floats: B=%d L=%d d=%d depth=%d plan=%s" % (B, L, d, depth, pl.as_dict()))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(20)
    xt = torch.empty((B, L, d), dtype=torch.float32, device="cuda")
    xt.normal_(0.0, 0.1, generator=gen)
    xt[:, 0] = 0.0
    step = 500_000
    for lo in range(0, B, step):      # running sums along time, a slice of the batch at a time (bounded temporaries)
        torch.cumsum(xt[lo:lo + step], dim=1, out=xt[lo:lo + step])
    out = torch.full((B, gpu.sig_size(d, depth)), float("nan"), dtype=torch.float32, device="cuda")
    assert gpu.sig_compute(gpu.default_ctx(), xt, depth, 0, out) == gpu.SIG_OK
    torch.cuda.synchronize()
    assert bool(torch.isfinite(out).all())
    pick = np.concatenate([np.arange(0, 12), np.arange(B - 12, B),
                           np.sort(np.random.default_rng(8).choice(B, size=40, replace=False))])
    idx = torch.from_numpy(pick).cuda()
    x = xt[idx].cpu().numpy()
    assert_parity(out[idx].cpu().numpy(), oracle.signature(x, depth), x, depth, False)


@pytest.mark.parametrize("d,depth", [(5, 3), (3, 4), (6, 3), (4, 3), (7, 3), (3, 3), (2, 4), (2, 5), (2, 6), (3, 5)])
def test_stream_mode_auto_with_the_deeper_prefix_entries(gpu, oracle, d, depth):
    """Stream mode takes the entry behind the first small lane state when that one has fewer than 16 lanes per path."""
    for B, L in [(5, 40), (70, 23), (600, 12)]:
        rc, pl = gpu.sig_plan(gpu.default_ctx(), B, L, d, depth, 1)
        assert rc == gpu.SIG_OK
        x = workloads.brownian_paths(B, L, d, seed=5400 + 13 * B + L + d)
        check(gpu, oracle, x, depth, True, None, label="auto, stream, plan p=%d c=%d t=%d" % (pl.prefix_depth, pl.chunks, pl.threads))
        if pl.row_workgroups > 0:   # the call wrote its rows from registers: the plan's own mapping as well
            pl.row_workgroups = 0
            check(gpu, oracle, x, depth, True, pl, label="the entry itself")
