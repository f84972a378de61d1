"""Cases that the speed of this library is measured on: whole Partial FC training steps.

A case is one training step as a user's program makes it: `pfc_sample` draws the classes of the
step, forward/backward gives loss and gradients, the update changes the sampled rows of the centers
and of their momentum.  The program keeps a context, the centers, the momentum and the output
buffers, and calls the step again and again with the step number counting up.

Keys of a case:
  B, D, N      samples, feature dimension, classes
  r            sampling ratio (1e-9: only the classes of the batch, k = number of distinct labels)
  precision    "bf16" or "fp32" operands of the matrix products
  calls        "three":   pfc_sample, pfc_forward_backward, pfc_update
               "fused":   pfc_sample, pfc_forward_backward_update
               "options": pfc_sample, pfc_forward_backward_ex with the cosine margin, the cosine
                          filter and the two diagnostics, pfc_update
  alpha        exponent of the long-tailed (Zipf) label distribution, 0: uniform labels
  noalloc      the sample comes from pfc_sample_noalloc (no context)
  aligned      weight of the label's center in a feature: 0 as at the start of training (features
               and centers independent), above 0 as later on
"""
import math

import torch

from paper_2203_15565_amd import binding

_PRECISION = {"fp32": binding.PRECISION_FP32, "bf16": binding.PRECISION_BF16}
_SCALE, _LR, _MU = 64.0, 0.1, 0.9
_MARGIN, _COS_MARGIN, _FILTER = 0.5, 0.4, 0.4


def _case(name, B, D, N, r, precision="bf16", calls="three", alpha=1.2, noalloc=False, aligned=0.0):
    return {"name": name, "B": B, "D": D, "N": N, "r": r, "precision": precision, "calls": calls,
            "alpha": alpha, "noalloc": noalloc, "aligned": aligned}


def listed():
    return [
        # A laboratory-size problem in single precision: the step is all latency and launches.
        _case("tiny_fp32", 128, 512, 10_000, 0.1, precision="fp32", alpha=0.0),
        # A data set of about 93 thousand identities on one GPU: short kernels, many of them.
        _case("medium", 512, 512, 93_431, 0.1, alpha=1.1),
        # The same in single precision, for a user who compares runs or debugs.
        _case("medium_fp32", 512, 512, 93_431, 0.1, precision="fp32", calls="fused", alpha=1.1),
        # A compact embedding of a mobile-size network, sampler without a context.
        _case("narrow_d128", 256, 128, 85_742, 0.3, noalloc=True),
        # Odd sizes everywhere, cosine margin with filter and diagnostics, later in training.
        _case("ragged_options", 333, 192, 120_007, 0.13, calls="options", alpha=1.1, aligned=0.5),
        # 360 thousand identities, ordinary ratio, the one-call form.
        _case("large_fused", 1024, 512, 360_232, 0.1, calls="fused", alpha=1.1),
        # The same data without sampling: the full softmax that Partial FC is compared with.
        _case("large_full", 1024, 512, 360_232, 1.0, alpha=1.1),
        # A wide embedding, which takes the one-call form through two kernels.
        _case("wide_d1024", 768, 1024, 205_990, 0.1, calls="fused"),
        # Two million identities at the ratio of 0.1: the workload of the benchmark.
        _case("headline", 1024, 512, 2_059_906, 0.1),
        # The same with the one-call form.
        _case("headline_fused", 1024, 512, 2_059_906, 0.1, calls="fused"),
        # Ten million identities, the largest set of centers that is trained on one GPU here.
        _case("extreme_fused", 2048, 512, 10_000_000, 0.05, calls="fused"),
        # An enlarged batch against the classes of the batch alone.
        _case("batch16k", 16_384, 512, 2_059_906, 1e-9),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        D = rng.choice([512] * 6 + [64, 128, 192, 256, 256, 320, 384, 448, 640, 768, 896, 1024, 1024])
        batch_only = rng.random() < 0.12
        B = _log_int(rng, 2048, 16_384) if batch_only else _log_int(rng, 48, 4096)
        N = _log_int(rng, 8_000, 10_000_000)
        r = 1e-9 if batch_only else 1.0 if rng.random() < 0.1 else math.exp(
            rng.uniform(math.log(0.04), math.log(0.5)))
        c = {"B": B, "D": D, "N": N, "r": r,
             "precision": "fp32" if rng.random() < 0.2 else "bf16",
             "calls": rng.choice(["three", "three", "fused", "fused", "options"]),
             "alpha": rng.choice([0.0, 1.1, 1.2]),
             "noalloc": rng.random() < 0.15 and N <= 1 << 24 and math.ceil(r * N) >= B,
             "aligned": rng.choice([0.0, 0.0, 0.5])}
        if binding_limits(c) and _cost(c) <= most and 4 * N * D <= 4 * 10_000_000 * 512:
            return c


def binding_limits(case):
    """Whether the sampled set stays below what a context takes."""
    k = _sampled(case)
    return k < (1 << 24 if case["precision"] == "fp32" else 1 << 25)


def _sampled(case):
    """Classes of one step, or the most there can be where that depends on the labels."""
    return max(min(case["B"], case["N"]), min(math.ceil(case["r"] * case["N"]), case["N"]))


def work(case):
    """Three products of B x D x k; centers and momentum rows read and written once, features read
    and their gradient written once, the center gradient written and read where it crosses the
    calls, labels and ids."""
    B, D, k = case["B"], case["D"], _sampled(case)
    if k > case["r"] * case["N"] + 1:   # k = number of distinct labels: its expectation
        p = torch.arange(1, case["N"] + 1, dtype=torch.float64).pow_(-case["alpha"])
        k = -torch.expm1(B * torch.log1p(-p / p.sum() * (1.0 - 1e-12))).sum().item()
    rows = 4 + (0 if case["calls"] == "fused" else 2)   # W and v in and out; dW out and in
    return {"bytes": rows * 4.0 * k * D + 2 * 4.0 * B * D + 8.0 * B + 4.0 * B + 4.0 * k,
            "flops": 3 * 2.0 * B * D * k}


def _cost(case):
    """Seconds, roughly: only to keep drawn cases below the largest listed one."""
    B, D, k = case["B"], case["D"], _sampled(case)
    return 30.0 * k * D / 5e12 + 6.0 * B * D * k / (8e14 if case["precision"] == "bf16" else 8e13)


def tolerance(case):
    """Against the step in 64 bits the outputs are off (2-norm) by up to 8e-7 with fp32 operands;
    with bf16 operands by up to 1.5e-3 for D >= 512, 3.8e-3 at D = 128 and 5.3e-3 with features
    aligned to their centers at D = 192: the error of a cosine is that of D products of size 1/D,
    and the loss multiplies it by the scale.  Single entries of the momentum are off by up to 3e-5
    and 0.43: a center that is nobody's label often gets its whole gradient from one sample."""
    if case["precision"] == "fp32":
        return {"rel": 1e-5, "max": 1e-3}
    rel = 6e-3 * max(1.0, 512.0 / case["D"]) * (1.5 if case["aligned"] else 1.0)
    return {"rel": min(rel, 2e-2), "max": 0.9}


def _labels(case, g, dev):
    B, N = case["B"], case["N"]
    if not case["alpha"]:
        return torch.randint(0, N, (B,), generator=g, device=dev)
    cdf = torch.arange(1, N + 1, dtype=torch.float64, device=dev).pow_(-case["alpha"]).cumsum_(0)
    u = torch.rand(B, generator=g, device=dev, dtype=torch.float64) * cdf[-1]
    rank = torch.searchsorted(cdf, u).clamp_(max=N - 1)
    return torch.randperm(N, generator=g, device=dev)[rank]


def prepare(case, seed):
    dev = torch.device("cuda")
    B, D, N = case["B"], case["D"], case["N"]
    g = torch.Generator(device=dev).manual_seed(seed)
    labels = _labels(case, g, dev)
    features = torch.randn((B, D), generator=g, device=dev)
    weight = torch.randn((N, D), generator=g, device=dev).mul_(0.01)
    if case["aligned"]:
        center = torch.nn.functional.normalize(weight[labels], dim=1) * math.sqrt(D)
        features.mul_(1.0 - case["aligned"]).add_(center, alpha=case["aligned"])
    cap = binding.pfc_num_sampled(N, B, case["r"])
    st = {
        "case": case, "step": 0, "seed": seed,
        "ctx": binding.Context(N, D, B, case["r"], _PRECISION[case["precision"]]),
        "labels": labels, "features": features, "weight": weight,
        "momentum": torch.zeros_like(weight),
        "idx": torch.zeros(cap, dtype=torch.int32, device=dev),
        "labels_local": torch.zeros(B, dtype=torch.int32, device=dev),
        "loss": torch.zeros(1, device=dev),
        "dfeatures": torch.zeros((B, D), device=dev),
    }
    if case["calls"] != "fused":
        st["dweight"] = torch.zeros((cap, D), device=dev)
    if case["calls"] == "options":
        st["stats"] = torch.zeros(2, device=dev)
    return st


def run(st):
    case, ctx = st["case"], st["ctx"]
    step = st["step"]
    st["step"] = step + 1
    if case["noalloc"]:
        k = binding.pfc_sample_noalloc(st["labels"], case["N"], case["r"], st["seed"], step,
                                       st["idx"], st["labels_local"])
    else:
        k = ctx.pfc_sample(st["labels"], case["r"], st["seed"], step, st["idx"],
                           st["labels_local"])
    if case["calls"] == "fused":
        ctx.pfc_forward_backward_update(
            st["features"], st["weight"], st["momentum"], st["idx"], k, st["labels_local"],
            _SCALE, _MARGIN, _LR, _MU, st["loss"], st["dfeatures"])
    elif case["calls"] == "three":
        ctx.pfc_forward_backward(
            st["features"], st["weight"], st["idx"], k, st["labels_local"], _SCALE, _MARGIN,
            st["loss"], st["dfeatures"], st["dweight"])
        ctx.pfc_update(st["weight"], st["momentum"], st["idx"], k, st["dweight"], _LR, _MU)
    else:
        ctx.pfc_forward_backward_ex(
            st["features"], st["weight"], st["idx"], k, st["labels_local"], _SCALE, _COS_MARGIN,
            binding.MARGIN_COSFACE, _FILTER, st["loss"], st["dfeatures"], st["dweight"],
            st["stats"])
        ctx.pfc_update(st["weight"], st["momentum"], st["idx"], k, st["dweight"], _LR, _MU)
    return {n: st[n] for n in ("idx", "labels_local", "loss", "dfeatures", "dweight", "stats",
                               "weight", "momentum") if n in st}
