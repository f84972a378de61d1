"""Rounding of the long sums of the two backward products with fp32 operands.

All features are one vector and all centers another one orthogonal to it, so every entry of a gradient
is a sum of equal terms: the worst case of a running sum, whose roundings all go the same way inside a
power of two (16,384 of them in one chain come out up to 2e-4 off).  The sums run in pieces of 256
(dfeatures) and 512 (dweight) products, or, with the 256-tiles of large batches, in slices of at most 4096
that are added afterwards."""
import math

import numpy as np
import pytest
import torch

from paper_2203_15565_amd import binding

pytestmark = pytest.mark.gpu

U = 2.0 ** -24   # half an ulp


# samples, classes, D, products of one sum of dweight and of dfeatures without a break; backward tile, slices of the
# batch and of the classes that the call has on 256 compute units (tests/test_step_plan.py sees to it)
EQUAL = [
    (2_048, 16_000, 512, 512, 256, 128, 1, 4),          # in pieces
    (5_000, 20_000, 576, 512, 256, 128, 1, 1),
    (6_884, 21_623, 384, 512, 256, 64, 1, 1),
    (14_912, 3_225, 640, 512, 256, 64, 1, 1),
    (16_384, 3_000, 128, 512, 256, 128, 10, 2),
    (16_384, 15_000, 256, 4_096, 4_096, 256, 13, 8),    # in slices
    (16_384, 3_000, 256, 4_096, 4_096, 256, 10, 2),
]
INDEPENDENT = [
    (4_096, 33_000, 64, 128, 1, 8), (4_096, 8_000, 320, 128, 1, 3), (2_048, 16_000, 512, 128, 1, 4),
    (6_884, 21_623, 384, 64, 1, 1), (14_099, 2_330, 256, 256, 28, 4),
]


@pytest.mark.parametrize("B,k,D,piece_w,piece_x", [c[:5] for c in EQUAL])
def test_sums_of_equal_terms(B, k, D, piece_w, piece_x):
    s, m = 64.0, 1.5
    rng = np.random.default_rng(B + k)
    x, w = np.zeros(D, np.float32), np.zeros(D, np.float32)
    x[: D // 2] = rng.random(D // 2) + 0.5
    w[D // 2:] = rng.random(D // 2) + 0.5
    print("equal terms", B, k, D, flush=True)
    X = torch.from_numpy(x).cuda().repeat(B, 1)
    W = torch.from_numpy(w).cuda().repeat(k, 1)
    idx = torch.arange(k, dtype=torch.int32, device="cuda")
    yl = torch.zeros(B, dtype=torch.int32, device="cuda")      # every sample carries class 0
    loss = torch.zeros(1, device="cuda")
    dX, dW = torch.zeros_like(X), torch.zeros_like(W)
    ctx = binding.Context(k, D, B, 1.0, binding.PRECISION_FP32)
    ctx.pfc_forward_backward(X, W, idx, k, yl, s, m, loss, dX, dW)
    assert ctx.pfc_check() == binding.PFC_OK
    ctx.close()
    # 64 bits: all cosines are 0, exp(0) = 1, the label logit is s cos(pi/2 + m)
    x64, w64 = x.astype(np.float64), w.astype(np.float64)
    nx, nw = np.linalg.norm(x64), np.linalg.norm(w64)
    p = math.exp(-s * math.sin(m))
    l = k - 1 + p
    want_W = s / l * x64 / nx                                  # B equal terms of 1/B, rows 1 ..
    want_X = s / B * ((k - 1) / l + (p / l - 1) * math.cos(m)) * w64 / nw / nx

    def off(got, want):
        sel = want != 0
        g = got[:, torch.from_numpy(sel).cuda()].double().cpu().numpy()
        return float(np.max(np.abs(g / want[sel] - 1.0)))
    # a piece, the sum of the pieces, at most 64 slices, and 16 roundings of the factors
    assert off(dW[1:], want_W) <= (piece_w + B / piece_w + 64 + 16) * U
    # the label part takes cos(m) = 7 % of the sum away
    assert off(dX, want_X) <= (piece_x + k / piece_x + 64 + 16) * U / (1 - math.cos(m))
    assert (dX[:, : D // 2].abs().max() <= 1e-6 * dX.abs().max()).item()


# Independent terms: rounding t of a sum of n terms is off by up to U of what is there by then, sqrt(t / n) of the
# result.  A piece of 512 products takes 192 roundings, the pieces and slices are added to each other: U / sqrt(3)
# sqrt(192 / 2 + n / 512 / 2) rms, and three roundings of the factors: a bar of 4.5e-7 .. 4.6e-7.  (Sums of 4096
# products without a break 9.1e-7, the first form; of 2048 6.8e-7, the second; of 1024 5.0e-7, the third.)
@pytest.mark.parametrize("B,k,D", [c[:3] for c in INDEPENDENT])
def test_sums_of_independent_terms(B, k, D):
    s, m = 1.0, 0.5
    g = torch.Generator(device="cuda").manual_seed(k)
    X = torch.randn((B, D), generator=g, device="cuda")
    W = torch.randn((k, D), generator=g, device="cuda").mul_(0.01)
    yl = torch.randint(0, 16, (B,), generator=g, device="cuda").to(torch.int32)
    idx = torch.arange(k, dtype=torch.int32, device="cuda")
    loss = torch.zeros(1, device="cuda")
    dX, dW = torch.zeros_like(X), torch.zeros_like(W)
    print("independent terms", B, k, D, flush=True)
    ctx = binding.Context(k, D, B, 1.0, binding.PRECISION_FP32)
    ctx.pfc_forward_backward(X, W, idx, k, yl, s, m, loss, dX, dW)
    assert ctx.pfc_check() == binding.PFC_OK
    ctx.close()
    xn = torch.nn.functional.normalize(X.double(), dim=1)
    e = torch.exp(s * (xn @ torch.nn.functional.normalize(W.double(), dim=1).t()))
    label = yl.long()[:, None]
    theta = e.gather(1, label).log().div(s).clamp(-1.0, 1.0).acos()
    e.scatter_(1, label, torch.exp(s * torch.cos(theta + m)))
    want = ((s / B) * (e / e.sum(dim=1, keepdim=True))).t() @ xn       # rows that are nobody's label: 16 ..
    off = ((dW[16:].double() - want[16:]).norm() / want[16:].norm()).item()
    print("off", off, flush=True)
    assert off <= (math.sqrt(192 / 2 + B / 512 / 2) + 3) * U / math.sqrt(3.0)
