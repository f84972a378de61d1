"""Rounding of a single product of two fp32 operands of the backward launch, which multiplies their 16-bit planes.

One sample has features, the others' are zero: an entry of the center gradient off the labels is one product
E_j x_d and zeros.  E_j and x_d are not known to the last bit, but the matrix of their products has rank one: what
each entry is off from that is the rounding of its product."""
import math

import pytest
import torch

from paper_2203_15565_amd import binding

pytestmark = pytest.mark.gpu

U = 2.0 ** -24   # half an ulp


# 64-, 128- and 256-tiles, the class set of the one-kernel form
@pytest.mark.parametrize("B,k,D", [(1, 300, 512), (512, 9_344, 512), (4_096, 20_000, 512), (300, 36_000, 512)])
def test_one_rounding_to_a_product(B, k, D):
    g = torch.Generator(device="cuda").manual_seed(k)
    X = torch.zeros((B, D), device="cuda")
    X[B // 3] = torch.randn(D, generator=g, device="cuda")
    W = torch.randn((k, D), generator=g, device="cuda")
    idx = torch.arange(k, dtype=torch.int32, device="cuda")
    yl = torch.zeros(B, dtype=torch.int32, device="cuda")
    loss = torch.zeros(1, device="cuda")
    dX, dW = torch.zeros_like(X), torch.zeros_like(W)
    print("products", B, k, D, flush=True)
    ctx = binding.Context(k, D, B, 1.0, binding.PRECISION_FP32)
    ctx.pfc_forward_backward(X, W, idx, k, yl, 16.0, 0.5, loss, dX, dW)
    assert ctx.pfc_check() == binding.PFC_OK
    ctx.close()
    p = dW[1:].double()
    x = p[0].clone()
    for _ in range(4):   # the factors, as means over many rounded products
        e = (p / x).mean(dim=1, keepdim=True)
        x = (p / e).mean(dim=0)
    off = ((p / (e * x) - 1.0) ** 2).mean().sqrt().item()
    print("off", off, flush=True)
    # a rounding is off by up to U of the power of two below the product: U / sqrt(3) rms at most, 0.74 of that over a
    # decade of mantissas; products of planes left out come to 2^-26 at most.  (The largest product of planes added
    # up first, and five more behind it: 5e-8.)
    assert off <= U / math.sqrt(3.0)
