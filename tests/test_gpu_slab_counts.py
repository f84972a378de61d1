"""The GEMM main loops at their shortest reductions, for every size of tile: fewer slabs than they hold in LDS,
exactly as many, and the first counts at which buffers are used again; fp32 operands of any size."""
import numpy as np
import pytest

from oracle import pfc_oracle as O

from paper_2203_15565_amd import binding
from pfc_harness import gpu_forward_backward, row_rel_max
from test_gpu_fused import test_fused_equals_two_calls as fused_equals_two_calls
from test_gpu_step import _fb_parity

pytestmark = pytest.mark.gpu

BF16, FP32 = binding.PRECISION_BF16, binding.PRECISION_FP32


# logits: D / 64 slabs; dweight: as many as 64 samples go into the padded batch; dfeatures: slices of at least 4
# (classes, samples, D, tiles of the logits and of the backward launch in bf16 and in fp32;
# tests/test_step_plan.py holds the rules to them; 128-tiles of the backward launch in bf16 at D = 64 and 128:
# BF16_FORMS of test_gpu_backward_launch.py)
FORMS = ([(1_000, 100, D, (64, 64), (64, 64)) for D in (64, 128, 192, 256, 320, 384)] +
         [(10_000, 300, D, (128, 64), (128, 64)) for D in (64, 128)] +
         [(10_000, 300, D, (128, 128), (128, 128)) for D in (192, 256, 320, 384)] +
         [(16_384, 1_024, 320, (256, 128), (256, 128)), (51_200, 256, 512, (128, 256), (64, 128)),
          (20_000, 512, 448, (128, 256), (64, 128))])


@pytest.mark.parametrize("N,B,D,bf16,fp32", FORMS)
@pytest.mark.parametrize("precision", [BF16, FP32])
def test_few_slabs(precision, N, B, D, bf16, fp32):
    _fb_parity(precision, N, B, D, 1.0, 64.0, 0.5, N + B + D)


# fused: slabs of 32 samples, four to eight of them; half-height tiles: of 64
@pytest.mark.parametrize("precision", [BF16, FP32])
@pytest.mark.parametrize("B", [48, 130, 256])
def test_few_slabs_fused(precision, B):
    fused_equals_two_calls(36_000, B, 512, 1.0, precision, 36_000, False)


# The fp32 operands of the backward products are split into 16-bit planes.  Rows of one component, of components 2^-40
# .. 1 and of equal ones; tolerances: a cosine is off by 2^-23 of its products, < 1.2e-7, the logit by 64 of that.
@pytest.mark.parametrize("N,B", [(300, 70), (5_000, 300), (33_000, 512)])
def test_fp32_components_of_any_size(N, B):
    import torch
    D, s, m = 512, 64.0, 0.5
    rng = np.random.default_rng(N)

    def rows(n):
        r = rng.standard_normal((n, D)) * 2.0 ** rng.uniform(-40.0, 0.0, (n, D))
        r[::3] = 0.0
        r[np.arange(0, n, 3), rng.integers(0, D, len(r[::3]))] = 7.0
        r[1::3] = rng.choice([-0.25, 0.25], (len(r[1::3]), D))
        return r.astype(np.float32)
    X, W = rows(B), rows(N)
    yl = rng.integers(0, N, B).astype(np.int32)
    idx = np.arange(N, dtype=np.int32)
    print("components", N, B, flush=True)
    ctx = binding.Context(N, D, B, 1.0, FP32)
    loss, dX, dWn = gpu_forward_backward(ctx, X, torch.from_numpy(W).cuda(), idx, yl, s, m)
    assert ctx.pfc_check() == binding.PFC_OK
    ctx.close()
    o = O.forward_backward(X, W, yl, s, m)
    assert abs(loss - o["loss"]) <= 1e-5 * abs(o["loss"])
    assert row_rel_max(dWn, o["dWn"])[0] <= 1e-4
    assert row_rel_max(dX, o["dX"])[0] <= 1e-4
