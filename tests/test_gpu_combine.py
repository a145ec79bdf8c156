"""The compiled product of dense rows (csrc/sig_combine.hip) over every shape it takes, against the general kernels: a batch of
at least 256 rows takes the compiled kernel, its pieces of fewer rows the others, which test_gpu_parity.py holds against
the oracle.  Rows of every length modulo four, ragged last workgroups, and operands that start off a 16-byte boundary."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHAPES = ([(d, 2) for d in range(2, 21)] + [(d, 3) for d in range(2, 17)] + [(d, 4) for d in range(2, 11)]
          + [(d, 5) for d in range(2, 7)] + [(d, 6) for d in range(2, 5)])


def product(binding, a, b, d, depth, out):
    rc = binding.sig_combine(binding.default_ctx(), a, b, d, depth, out)
    assert rc == binding.SIG_OK, rc
    return out


@pytest.mark.parametrize("d,depth", SHAPES, ids=lambda v: str(v))
def test_every_compiled_shape_against_the_general_kernels(d, depth):
    """Each word is a sum of depth + 1 terms in two orders: the two differ by at most 2 (depth + 1) 2^-24 of the sum of
    the terms' magnitudes, which is the same product of the operands' magnitudes."""
    import torch
    from paper_2501_08455_amd import binding
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    D = binding.sig_size(d, depth)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(100 * d + depth)
    # 256 rows: one row to a workgroup; the others several, with a ragged last workgroup
    for B, shift in ((256, 0), (257, 1), (2051, 3), (8195, 2)):
        if B * D > 12_000_000:
            continue
        print("product of %d rows of (%d,%d), operands %d floats off" % (B, d, depth, shift), flush=True)
        a, b, out = (torch.randn(B * D + 4, device="cuda", generator=gen)[s:s + B * D].view(B, D) for s in (shift, 0, shift))
        out.fill_(float("nan"))
        product(binding, a, b, d, depth, out)
        step = 255
        for lo in range(0, B, max(step, (B // 4 // step) * step)):
            hi = min(lo + step, B)
            want = product(binding, a[lo:hi], b[lo:hi], d, depth, torch.empty_like(a[lo:hi]))
            size = product(binding, a[lo:hi].abs(), b[lo:hi].abs(), d, depth, torch.empty_like(want))
            worst = float(((out[lo:hi] - want).abs() / size).max())
            assert np.isfinite(worst) and worst <= 2 * (depth + 1) * 2.0 ** -24, (B, lo, worst)
        assert bool(torch.isfinite(out).all())


def test_infinite_and_undefined_coefficients_stay_where_they_belong():
    import torch
    from paper_2501_08455_amd import binding
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    d, depth, B = 5, 4, 300
    D = binding.sig_size(d, depth)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    a, b = torch.randn((B, D), device="cuda", generator=gen), torch.randn((B, D), device="cuda", generator=gen)
    a[3, 2], a[4, 29], b[5, 154], b[299, D - 1] = float("inf"), float("nan"), float("-inf"), float("nan")
    got = product(binding, a, b, d, depth, torch.empty_like(a))
    for lo in (0, 150):
        want = product(binding, a[lo:lo + 150], b[lo:lo + 150], d, depth, torch.empty_like(a[:150]))
        part = got[lo:lo + 150]
        assert torch.equal(torch.isnan(part), torch.isnan(want)) and torch.equal(torch.isinf(part), torch.isinf(want))
