"""The work whose speed this library answers for: listed cases, and draws from the ranges they stand for.

Every case is one call (or one forward/backward pair) through the Python entry points a program uses:
`binding.signature`, `autograd.signature` with `torch.autograd.grad`, and `binding.sig_combine`.  Inputs are made on the
GPU from a seed; path laws are those of `workloads.py` (Brownian increments N(0, 1/L), or uniform ones for the large
signature).  All data is float32, the only type the library takes.

A case is {"op", "B", "L", "d", "depth", "stream", "law"}; "combine" has no L, stream or law.
"""
import math

import torch

from paper_2501_08455_amd import autograd, binding, workloads


def _case(op, B, L, d, depth, stream=False, law="normal", name=None):
    c = {"op": op, "B": B, "d": d, "depth": depth}
    if op != "combine":
        c.update(L=L, stream=stream, law=law)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # a handful of short two-channel paths: an interactive call, all launch and host latency
        _case("forward", 4, 16, 2, 3, name="tiny_forward"),
        # one mini-batch of the paper's comparison tables: inference on a batch
        _case("forward", 128, 100, 5, 4, name="batch_forward"),
        # the same batch with long series: the time-parallel scan
        _case("forward", 128, 2000, 5, 4, name="long_forward"),
        # every prefix of a mini-batch: the layer in front of a sequence model
        _case("forward", 64, 256, 4, 4, stream=True, name="stream_forward"),
        # ten channels at depth six: few paths, 1.1 million coefficients each
        _case("forward", 16, 128, 10, 6, law="uniform", name="large_forward"),
        # features of a whole data set in one call
        _case("forward", 65536, 100, 5, 4, name="bulk_forward"),
        # the signature layer of one training step, forward and backward
        _case("train", 128, 100, 5, 4, name="train_step"),
        # the ragged last batch of an epoch (12,765 samples in batches of 128) of longer series
        _case("train", 93, 500, 4, 4, name="train_ragged"),
        # one step on more channels than the register kernels take
        _case("train", 128, 100, 12, 3, name="train_wide"),
        # full-batch training on a whole data set
        _case("train", 65536, 100, 5, 4, name="train_bulk"),
        # sequence-to-sequence training on a large batch: every prefix has an upstream gradient
        _case("train", 4096, 256, 4, 4, stream=True, name="train_stream_bulk"),
        # Chen's identity on two batches of signatures: windows joined without going back to the paths
        _case("combine", 65536, 0, 5, 4, name="combine_bulk"),
    ]


# (channels, depth) a program asks for: two to ten channels while a row stays within some ten thousand coefficients, and
# more channels at the depths that are affordable there
_SHAPES = [(d, n) for d in range(2, 11) for n in range(2, 7) if workloads.sig_size(d, n) <= 12000]
_WIDE = [(d, 2) for d in range(11, 21)] + [(11, 3), (12, 3)]

# one drawn case moves and computes no more than the largest listed ones
_MOST_BYTES = 2.87e9
_MOST_FLOPS = 3.78e10


def _log_uniform(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(("forward", "forward", "forward", "train", "train", "train", "combine"))
    d, depth = rng.choice(_WIDE if rng.random() < 0.15 else _SHAPES)
    if op == "combine":
        case = _case(op, _log_uniform(rng, 1, 65536), 0, d, depth)
        most = 2.5 * 65536 * 780
        case["B"] = max(1, min(case["B"], int(most / workloads.sig_size(d, depth))))
        return case
    L = _log_uniform(rng, 8, 2000)
    B = _log_uniform(rng, 1, 65536)
    stream = rng.random() < 0.4
    law = "uniform" if L <= 256 and rng.random() < 0.3 else "normal"
    if rng.random() < 0.08:
        # the large signature: few paths
        return _case(op, _log_uniform(rng, 1, 16), _log_uniform(rng, 16, 128), 10, 6, law="uniform")
    if op == "train" and d > 10:
        # training batches of short series, as in the listed case
        L = _log_uniform(rng, 8, 150)
        B = _log_uniform(rng, 1, 128)
    case = _case(op, B, L, d, depth, stream=stream, law=law)
    w = work(case)
    over = max(w["bytes"] / _MOST_BYTES, w["flops"] / _MOST_FLOPS)
    if over > 1.0:
        case["B"] = max(1, int(B / over))
    return case


def _paths(case, gen):
    """float32 paths from 0 with i.i.d. increments, summed in float64 and rounded once."""
    B, L, d = case["B"], case["L"], case["d"]
    x = torch.zeros((B, L, d), dtype=torch.float64, device="cuda")
    inc = x[:, 1:, :]
    if case["law"] == "normal":
        inc.normal_(0.0, math.sqrt(1.0 / L), generator=gen)
    else:
        inc.uniform_(-0.1, 0.1, generator=gen)
    return x.cumsum(1).float()


def _rows(case, gen):
    """Rows with the spread of Brownian signatures on [0, 1]: a coefficient of level n has variance about 1/n!."""
    levels = [torch.randn((case["B"], case["d"] ** n), device="cuda", generator=gen) / math.sqrt(math.factorial(n))
              for n in range(1, case["depth"] + 1)]
    return torch.cat(levels, dim=1)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    state = dict(case)
    if case["op"] == "combine":
        state["a"], state["b"] = _rows(case, gen), _rows(case, gen)
        state["out"] = torch.empty_like(state["a"])
        state["ctx"] = binding.default_ctx()
        return state
    state["path"] = _paths(case, gen)
    if case["op"] == "train":
        B, K, D = case["B"], case["L"] - 1, workloads.sig_size(case["d"], case["depth"])
        shape = (B, K, D) if case["stream"] else (B, D)
        state["grad_out"] = torch.randn(shape, device="cuda", generator=gen)
        state["path"].requires_grad_(True)
    return state


def run(state):
    op = state["op"]
    if op == "forward":
        return binding.signature(state["path"], state["depth"], stream=state["stream"])
    if op == "train":
        out = autograd.signature(state["path"], state["depth"], stream=state["stream"])
        (grad,) = torch.autograd.grad(out, state["path"], state["grad_out"])
        return out, grad
    rc = binding.sig_combine(state["ctx"], state["a"], state["b"], state["d"], state["depth"], state["out"])
    if rc != binding.SIG_OK:
        raise binding.SigError(rc, "sig_combine")
    return state["out"]


def work(case):
    B, d, depth = case["B"], case["d"], case["depth"]
    D = workloads.sig_size(d, depth)
    if case["op"] == "combine":
        # level n is a sum of n - 1 outer products and the two factors' own levels
        return {"bytes": 4.0 * 3 * B * D, "flops": 2.0 * B * sum(n * d ** n for n in range(1, depth + 1))}
    K = case["L"] - 1
    rows = K if case["stream"] else 1
    step = 2.0 * workloads.fused_fma_per_step(d, depth)
    nbytes, flops = 4.0 * (B * case["L"] * d + B * rows * D), step * B * K
    if case["op"] == "train":
        # backward: the upstream gradient in, the gradient of the path out, two multiply-adds for each of the forward
        nbytes += 4.0 * (B * case["L"] * d + B * rows * D)
        flops *= 3.0
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # rounding of float32 sums over K increments folded one after the other, two implementations apart
    K = case["L"] - 1 if case["op"] != "combine" else 1
    return {"rel": max(1e-5, 4e-7 * math.sqrt(K))}
