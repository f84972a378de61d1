"""The label part of batches of several windows, where the number of a class's samples in a window matters: one
wavefront sums up to 8, all wavefronts of a workgroup more, up to a whole window of 1024."""
import numpy as np
import pytest

from oracle import pfc_oracle as O
from paper_2203_15565_amd import binding
from pfc_harness import ROW_GRAD_TOL, gpu_forward_backward, gpu_sample, rel_max, row_rel_max

pytestmark = pytest.mark.gpu

N = 3000
COUNTS = [1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 18, 31, 32, 33, 64, 65, 200]   # samples of one class in a window


def _labels(B, rng):
    """Window 0 all one class (N - 1, the last of the sorted ones); the others COUNTS and single samples,
    shuffled; a last window may hold a few samples only."""
    y = np.full(B, N - 1, dtype=np.int64)
    for w0 in range(1024, B, 1024):
        n = min(1024, B - w0)
        part = np.repeat(rng.permutation(N)[: len(COUNTS)], COUNTS)[:n]
        part = np.concatenate([part, rng.integers(0, N, size=n - part.size)])
        y[w0:w0 + n] = rng.permutation(part)
    return y


@pytest.mark.parametrize("B", [1025, 2048, 3100])
@pytest.mark.parametrize("D", [64, 320, 768, 1024])
def test_class_sizes_in_a_window(B, D):
    import torch
    print("label windows", B, D, flush=True)
    rng = np.random.default_rng(B + D)
    X = rng.standard_normal((B, D)).astype(np.float32)
    W = (rng.standard_normal((N, D)) * 0.01).astype(np.float32)
    labels = _labels(B, rng)
    ctx = binding.Context(N, D, B, 0.3, binding.PRECISION_FP32)
    idx, yl, k = gpu_sample(ctx, labels, 0.3, 0, 0)
    idx = idx[:k]
    Wd = torch.from_numpy(W).cuda()
    loss, dX, dW = gpu_forward_backward(ctx, X, Wd, idx, yl, 64.0, 0.5)
    o = O.forward_backward(X, W[idx.astype(np.int64)], yl, 64.0, 0.5)
    # bars of the fp32 parity tests: the rounding of a cosine times the scale; sums of 1024 rows add less
    assert rel_max(dW, o["dWn"]) <= 2e-5
    assert row_rel_max(dW, o["dWn"])[0] <= ROW_GRAD_TOL[binding.PRECISION_FP32]
    assert rel_max(dX, o["dX"]) <= 2e-5
    again = gpu_forward_backward(ctx, X, Wd, idx, yl, 64.0, 0.5)
    assert again[1].tobytes() == dX.tobytes() and again[2].tobytes() == dW.tobytes()
    ctx.close()
