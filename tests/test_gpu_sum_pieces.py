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


# 128-tiles with the batch in one slice, 64-tiles, 128-tiles with the batch cut into slices: in pieces.
# 256-tiles: the classes in four slices, or the batch in many.
@pytest.mark.parametrize("B,k,D,piece_w,piece_x", [
    (2_048, 16_000, 512, 512, 256), (4_096, 33_000, 64, 512, 256), (16_384, 3_000, 128, 512, 256),
    (16_384, 15_000, 256, 4_096, 4_096), (16_384, 3_000, 256, 4_096, 4_096)])
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
