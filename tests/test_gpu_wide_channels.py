"""The on-chip kernels of more than ten channels (csrc/sig_onchip_table_wide.hip), every compiled shape in final mode against
the fp64 oracle: whole paths side by side with a ragged last workgroup, chunks of a path side by side, and paths cut
across workgroups, with lengths that leave remainders.  The gate is the library's 1e-4 per level."""
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
        rows = sorted({0, 1, 7, B // 2, B - 2, B - 1})
        got, want = out[rows].cpu().numpy().astype(np.float64), oracle.signature(x[rows], depth)
        start = 0
        for n in range(1, depth + 1):
            sl = slice(start, start + d ** n)
            err = np.linalg.norm(got[:, sl] - want[:, sl], axis=1) / np.linalg.norm(want[:, sl], axis=1)
            assert float(err.max()) <= 1e-4, (B, L, n, float(err.max()))
            start += d ** n
