"""The fp32 logits of few 64-tiles (64 classes x 16 samples to a workgroup): parity at the edges of its tiles and
stages, and the bits of the 64-tiles."""
import numpy as np
import pytest

from paper_2203_15565_amd import binding
from test_gpu_options import _run_ex
from test_gpu_step import _fb_parity

pytestmark = pytest.mark.gpu

FP32 = binding.PRECISION_FP32


# stages of 64 columns: 1, 3, 4, 5, 16; classes: part of a tile, one more than a tile, the most there are (128 tiles
# where half of 256 compute units are full); samples: 1, either side of 16 and 64
# (tests/test_step_plan.py holds the rule to what is said here)
SLIM = [(40, 1, 64), (65, 15, 192), (300, 16, 256), (1000, 17, 320), (1000, 65, 1024), (8192, 64, 512), (4096, 128, 64)]


@pytest.mark.parametrize("N,B,D", SLIM)
def test_parity(N, B, D):
    # (with few samples a large scale leaves most rows of dWn below the floor of the row bar)
    _fb_parity(FP32, N, B, D, 1.0, 64.0 if B >= 64 else 10.0, 0.5, N + B + D)
    if B >= 64:   # the largest logit of every sample first
        _fb_parity(FP32, N, B, D, 1.0, 100.0, 0.5, N + B + D, dup=True)


def test_options():
    _run_ex(FP32, 3000, 40, 192, 0.5, 64.0, 0.4, "cosface", 0.4, seed=5, clusters=3)
    _run_ex(FP32, 2000, 17, 512, 1.0, 160.0, 0.3, "arcface", 0.35, seed=6, clusters=3)


# Copies of one sample: the mean loss is the loss of each, the means of the cosines are the cosines.  8192 classes are
# 128 tiles for 64 samples and 256 for 128, which take the 64-tiles.
@pytest.mark.parametrize("D,aligned", [(64, 0.0), (512, 0.0), (512, 0.6), (832, 0.8)])
def test_bits_of_the_64_tiles(D, aligned):
    import torch
    N = 8192
    rng = np.random.default_rng(D)
    W = rng.standard_normal((N, D)).astype(np.float32)
    Wd = torch.from_numpy(W).cuda()
    idx = torch.arange(N, dtype=torch.int32, device="cuda")
    for y in (0, 37, 4095, N - 1):
        w = W[y] / np.linalg.norm(W[y]) * np.sqrt(D)
        x = (rng.standard_normal(D) * (1.0 - aligned) + w * aligned).astype(np.float32)
        out = []
        for B in (64, 128):
            print("bits", D, aligned, y, B, flush=True)
            ctx = binding.Context(N, D, B, 1.0, FP32)
            loss, stats = torch.zeros(1, device="cuda"), torch.zeros(2, device="cuda")
            X = torch.from_numpy(np.tile(x, (B, 1))).cuda()
            dX, dW = torch.zeros(B, D, device="cuda"), torch.zeros(N, D, device="cuda")
            ctx.pfc_forward_backward_ex(X, Wd, idx, N, torch.full((B,), y, dtype=torch.int32, device="cuda"), 64.0, 0.5,
                                        binding.MARGIN_ARCFACE, 2.0, loss, dX, dW, stats)
            torch.cuda.synchronize()
            out.append(torch.cat([loss, stats]).cpu())
            ctx.close()
        assert torch.equal(out[0], out[1]), out
