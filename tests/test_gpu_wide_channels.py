"""The on-chip kernels of more than ten channels (csrc/sig_onchip_table_wide.hip), every compiled shape in final mode against
the fp64 oracle: whole paths side by side with a ragged last workgroup, chunks of a path side by side, and paths cut
across workgroups, with lengths that leave remainders; then every form of a plan that sig_compute_planned accepts for them.
The gate is the library's 1e-4 per level."""
import numpy as np
import pytest

from paper_2501_08455_amd import binding, workloads

SHAPES = [(d, 2) for d in range(11, 21)] + [(d, 3) for d in (11, 12)]


@pytest.mark.parametrize("d,depth", SHAPES, ids=lambda v: str(v))
def test_planner_takes_the_compiled_kernel(d, depth):
    for B, L in [(16, 2), (128, 100), (93, 501), (65536, 20)]:
        rc, pl = binding.sig_plan(None, B, L, d, depth, 0)
        assert rc == binding.SIG_OK and (pl.variant, pl.prefix_depth) == (binding.SIG_VARIANT_ON_CHIP, depth - 1)
        assert binding.sig_plan_validate(B, L, d, depth, 0, pl) == binding.SIG_OK


@pytest.mark.parametrize("d,depth", SHAPES, ids=lambda v: str(v))
def test_stream_mode_refuses_the_compiled_kernel(d, depth):
    """As the planner does not take it there, no explicit plan may ask for it."""
    for B, L in [(1, 2), (17, 40), (4096, 100)]:
        rc, pl = binding.sig_plan(None, B, L, d, depth, 1)
        assert rc == binding.SIG_OK and pl.variant == binding.SIG_VARIANT_LEVEL_SCAN
        for chunks in (1, 2, 4):
            for waves in (0, 1):
                plan = binding.make_plan(binding.SIG_VARIANT_ON_CHIP, prefix_depth=depth - 1, chunks=chunks, independent_waves=waves)
                assert binding.sig_plan_validate(B, L, d, depth, 1, plan) == binding.SIG_ERR_INVALID
                assert binding.sig_plan_footprint(B, L, d, depth, 1, plan)[0] == binding.SIG_ERR_INVALID


@pytest.mark.gpu
@pytest.mark.parametrize("d,depth", SHAPES, ids=lambda v: str(v))
def test_against_the_oracle(oracle, d, depth):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    for B, L in [(17, 2), (128, 100), (93, 151), (16, 1003), (8195, 13)]:
        print("wide forward: %d paths of %d points, (%d,%d)" % (B, L, d, depth), flush=True)
        x = workloads.brownian_paths(B, L, d, seed=9400 + d + L)
        out = torch.full((B, binding.sig_size(d, depth)), float("nan"), device="cuda")
        assert binding.sig_compute(binding.default_ctx(), torch.from_numpy(x).cuda(), depth, 0, out) == binding.SIG_OK
        assert bool(torch.isfinite(out).all())
        check_rows(oracle, x, out, d, depth, (B, L))


@pytest.mark.gpu
@pytest.mark.parametrize("d,depth,B,L,paths", [(12, 3, 300, 1100, 24), (12, 3, 16, 4000, 8), (11, 3, 700, 2500, 8), (20, 2, 14000, 1500, 64), (13, 2, 30000, 1027, 64)])
def test_long_paths_in_eight_pieces_and_more(oracle, d, depth, B, L, paths):
    """Beyond 128 steps a piece, or by chunks where the batch alone fills the chip: against the oracle, and no further from it than one
    launch per level, which summed the whole path in one go (measured 0.2 to 0.75 of its error)."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    rc, pl = binding.sig_plan(None, B, L, d, depth, 0)
    assert rc == binding.SIG_OK and pl.variant == binding.SIG_VARIANT_ON_CHIP and pl.chunks * pl.segments >= 8
    print("wide forward, long: %d paths of %d points, (%d,%d)" % (B, L, d, depth), flush=True)
    x = torch.zeros((B, L, d), device="cuda")
    x[:, 1:].normal_(0.0, L ** -0.5, generator=torch.Generator(device="cuda").manual_seed(d + L))
    x = x.cumsum(1)
    out = torch.full((B, binding.sig_size(d, depth)), float("nan"), device="cuda")
    assert binding.sig_compute(binding.default_ctx(), x, depth, 0, out) == binding.SIG_OK
    assert bool(torch.isfinite(out).all())
    pick = np.unique(np.linspace(0, B - 1, paths).astype(int))
    idx = torch.from_numpy(pick).cuda()
    few = x[idx].contiguous()
    want = oracle.signature(few.cpu().numpy(), depth)
    level = torch.empty((len(pick), out.shape[1]), device="cuda")
    plan = binding.make_plan(binding.SIG_VARIANT_LEVEL_SCAN, chunks=1 if B * d ** (depth - 1) > 200000 else 0)
    assert binding.sig_compute(binding.default_ctx(), few, depth, 0, level, plan=plan) == binding.SIG_OK
    error = lambda y: np.linalg.norm(y.cpu().numpy() - want) / np.linalg.norm(want)   # noqa: E731
    print("  rel err %.2e, level by level %.2e" % (error(out[idx]), error(level)))
    assert error(out[idx]) <= 1e-4 and error(out[idx]) <= 1.1 * error(level)


def check_rows(oracle, x, out, d, depth, label):
    B = x.shape[0]
    rows = sorted({0, 1, 7, B // 2, B - 2, B - 1} & set(range(B)))
    got, want = out[rows].cpu().numpy().astype(np.float64), oracle.signature(x[rows], depth)
    start = 0
    for n in range(1, depth + 1):
        sl = slice(start, start + d ** n)
        err = np.linalg.norm(got[:, sl] - want[:, sl], axis=1) / np.linalg.norm(want[:, sl], axis=1)
        assert float(err.max()) <= 1e-4, (label, n, float(err.max()))
        start += d ** n


# fields of a plan; the ones a shape cannot hold (more chunks than its lanes leave room for) are refused by the host checks
FORMS = [dict(), dict(independent_waves=1), dict(independent_waves=1, tile_steps=5), dict(tile_steps=7, tile_loader=1),
         dict(tile_steps=7, tile_loader=2), dict(chunks=2, threads=512), dict(chunks=3, tile_steps=4, tile_loader=1),
         dict(chunks=3, tile_steps=4, tile_loader=2), dict(segments=2), dict(segments=3, chunks=2, threads=512), dict(segments=4),
         dict(segments=16), dict(threads=192), dict(stagger_ticks=50)]


@pytest.mark.gpu
@pytest.mark.parametrize("d,depth", SHAPES, ids=lambda v: str(v))
def test_explicit_plans_against_the_oracle(oracle, d, depth):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    ctx, ran = binding.default_ctx(), 0
    for B, L in [(3, 70), (131, 41)]:
        x = workloads.brownian_paths(B, L, d, seed=9700 + d + L)
        path = torch.from_numpy(x).cuda()
        for form in FORMS:
            plan = binding.make_plan(binding.SIG_VARIANT_ON_CHIP, prefix_depth=depth - 1, **form)
            out = torch.full((B, binding.sig_size(d, depth)), float("nan"), device="cuda")
            if binding.sig_plan_validate(B, L, d, depth, 0, plan) != binding.SIG_OK:
                assert binding.sig_compute(ctx, path, depth, 0, out, plan=plan) == binding.SIG_ERR_INVALID, form
                continue
            print("explicit plan: %d paths of %d points, (%d,%d), %s" % (B, L, d, depth, form), flush=True)
            assert binding.sig_compute(ctx, path, depth, 0, out, plan=plan) == binding.SIG_OK, form
            assert bool(torch.isfinite(out).all()), form
            check_rows(oracle, x, out, d, depth, (B, L, form))
            ran += 1
    assert ran >= 12


@pytest.mark.gpu
@pytest.mark.parametrize("d,depth,B,L,stream", [(12, 3, 4, 30, 0), (20, 2, 9, 200, 0), (11, 3, 9, 40, 1), (16, 2, 5, 60, 1)])
def test_tuned_plans(oracle, d, depth, B, L, stream):
    """What sig_autotune settles on, with fewer paths than the planner asks for and in stream mode."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    ctx = binding.sig_create()
    try:
        x = workloads.brownian_paths(B, L, d, seed=9800 + d)
        rc, plan, _ = binding.sig_autotune(ctx, B, L, d, depth, stream)
        assert rc == binding.SIG_OK and (not stream or plan.variant != binding.SIG_VARIANT_ON_CHIP)
        D = binding.sig_size(d, depth)
        out = torch.full((B, L - 1, D) if stream else (B, D), float("nan"), device="cuda")
        assert binding.sig_compute(ctx, torch.from_numpy(x).cuda(), depth, stream, out) == binding.SIG_OK
        got, want = out.cpu().numpy().astype(np.float64), oracle.signature(x, depth, stream=bool(stream))
        assert np.linalg.norm(got - want) <= 1e-4 * np.linalg.norm(want)
    finally:
        torch.cuda.synchronize()
        binding.sig_destroy(ctx)


@pytest.mark.gpu
def test_batches_whose_partial_rows_exceed_the_scratch_limit_go_in_slices(oracle):
    """150,001 paths of 900 points, (12,3): eight segments, 9.0 GB of partial rows, two slices.  Every path gives the bits that
    it gives in a batch of its own slice's neighbours under the same plan."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    B, L, d, depth = 150001, 900, 12, 3
    rc, plan = binding.sig_plan(None, B, L, d, depth, 0)
    assert rc == binding.SIG_OK and plan.variant == binding.SIG_VARIANT_ON_CHIP and plan.segments == 8
    D = binding.sig_size(d, depth)
    rc, _, _, scratch = binding.sig_plan_footprint(B, L, d, depth, 0, plan)
    S = scratch // (4 * plan.segments * D)
    assert rc == binding.SIG_OK and scratch <= 8 << 30 and S == 75001
    ctx = binding.sig_create()
    try:
        gen = torch.Generator(device="cuda").manual_seed(9900)
        path = torch.randn((B, L, d), device="cuda", generator=gen).mul_(L ** -0.5)
        torch.cumsum(path, 1, out=path)
        out = torch.full((B, D), float("nan"), device="cuda")
        assert binding.sig_compute(ctx, path, depth, 0, out) == binding.SIG_OK
        assert bool(torch.isfinite(out).all())
        for lo in (0, S - 40, B - 80):   # the ends, and across the border of the slices
            part = torch.empty((80, D), device="cuda")
            assert binding.sig_compute(ctx, path[lo:lo + 80], depth, 0, part, plan=plan) == binding.SIG_OK
            assert torch.equal(part, out[lo:lo + 80]), lo
            check_rows(oracle, path[lo:lo + 80].cpu().numpy(), part, d, depth, lo)
    finally:
        torch.cuda.synchronize()
        binding.sig_destroy(ctx)
