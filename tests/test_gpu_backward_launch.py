"""The two backward products share one launch, and the size of the GEMM tiles follows from the
problem: parity where the launch changes its shape -- from one tile size to the next, from one slice
of the classes to several, with the batch cut into slices, with a last slice shorter than the
others, and with batches and rows that end inside a tile."""
import numpy as np
import pytest
import torch

from oracle import pfc_oracle as O
from paper_2203_15565_amd import binding
from pfc_harness import gpu_forward_backward, gpu_sample, rel_max
from test_gpu_step import GRAD_TOL, LOSS_TOL, _fb_parity

pytestmark = pytest.mark.gpu

# (N, B, D, r)
CASES = [
    (32_512, 64, 256, 1.0),     # a whole number of tiles of 256 classes
    (32_513, 64, 256, 1.0),     # the last of them with one class
    (1_000, 64, 512, 0.256),    # one tile of 256 classes, one slice of dfeatures (fp32: two)
    (1_000, 64, 512, 0.257),    # two of them, twice the slices, the second tile with one class
    (6_000, 1_024, 64, 0.5),    # batch of a whole number of tiles, cut into slices; fp32: D narrower than a tile
    (50_000, 2_049, 320, 1e-9),  # classes of the batch alone: batch cut into slices
    (50_000, 4_096, 256, 1e-9),  # likewise, whole tiles
    (300, 65, 64, 1.0),         # 64-tiles, second tile of the batch with one sample, half a column tile
    (16_384, 128, 128, 1.0),    # bf16: 128 tiles of 128 classes: 64-tiles for logits and backward
    (16_385, 129, 128, 1.0),    # one more of each: bf16: 128-tiles for the logits
    (3_300, 512, 384, 1.0),     # six column tiles of 64
    (16_000, 1_024, 320, 1.0),  # 256-tiles for the logits alone (0.98 of a round), rows of 384
    (16_000, 1_000, 512, 1.0),  # the same, batch ends inside a tile
    (9_000, 300, 640, 1.0),     # fp32: 64-tiles, bf16: 128-tiles; five column tiles
    (8_192, 256, 512, 1.0),     # fp32: exactly one 128-tile per compute unit
    # batches above 2048, 256-tiles in both precisions:
    (3_000, 8_100, 512, 1.0),   # batch and classes cut, dweight in front, last slices shorter, batch ends inside a tile
    (16_100, 4_000, 512, 1.0),  # batch in one piece, dweight in front
    (2_000, 4_096, 768, 1.0),   # dfeatures in front; three column tiles
    (5_000, 2_250, 1_024, 1.0),  # bf16: batch in one piece
]


@pytest.mark.parametrize("N,B,D,r", CASES)
@pytest.mark.parametrize("precision", [binding.PRECISION_FP32, binding.PRECISION_BF16])
def test_backward_launch_edges(precision, N, B, D, r):
    _fb_parity(precision, N, B, D, r, 64.0, 0.5, seed=5)


# bf16 forms at sizes where a kernel can go wrong: (N, B, D, tiles of the logits and of the backward launch, slices of
# the batch and of the classes); tests/test_step_plan.py holds the rules to them.  (256-tiles with the batch cut
# are for batches above 2048 alone: 3,000 x 8,100 and 2,000 x 4,096 above.)
BF16_FORMS = [
    (20_000, 137, 64, 128, 128, 1, 32),     # 128-tiles, half a column tile, shortest reductions
    (19_000, 137, 128, 128, 128, 1, 30),    # one column tile
    (16_385, 129, 192, 128, 128, 1, 26),    # a tile and one sample, a tile and one class
    (233, 1_430, 384, 64, 128, 3, 1),       # three column tiles of 128, batch cut, one slice of dfeatures
    (9_345, 300, 384, 128, 128, 1, 14),     # three column tiles, classes cut
    (701, 1_186, 64, 64, 64, 2, 2),         # 64-tiles, batch and classes cut
    (21_487, 652, 448, 256, 256, 1, 14),    # 256-tiles everywhere, batch and columns end inside a tile
    (20_225, 726, 512, 256, 256, 1, 16),    # likewise, the last tile with one class
    (31_791, 910, 384, 256, 128, 1, 9),     # 256-tiles for the logits alone
]


@pytest.mark.parametrize("N,B,D,logits,backward,dw,dx", BF16_FORMS)
def test_bf16_forms(N, B, D, logits, backward, dw, dx):
    _fb_parity(binding.PRECISION_BF16, N, B, D, 1.0, 64.0 if B > 200 else 20.0, 0.5, seed=N + B)


# (N, B, D, r): the last launch (label parts, rows of dfeatures, loss) takes four samples to a
# workgroup, or one where the classes were cut into at least 12 slices and there is a compute unit
# for every sample.  Scale 16: with a few samples a peaked softmax leaves most
# rows of the center gradient below the floor of the row-wise bar.
FINAL_CASES = [
    (5_000, 1, 64, 0.01),       # one sample
    (5_000, 5, 1_024, 0.01),    # one sample in the second workgroup, few slices
    (40_000, 7, 1_024, 1.0),    # one sample to a workgroup
    (40_000, 1_023, 192, 0.5),  # last workgroup with three samples
    (40_000, 1_025, 192, 0.5),  # window sums of the label part, the second of one sample
    (20_000, 256, 192, 1.0),    # 12 slices and more: one sample to a workgroup (256 compute units) ..
    (20_000, 257, 192, 1.0),    # .. and four
]


@pytest.mark.parametrize("N,B,D,r", FINAL_CASES)
@pytest.mark.parametrize("precision", [binding.PRECISION_FP32, binding.PRECISION_BF16])
def test_final_launch_edges(precision, N, B, D, r):
    _fb_parity(precision, N, B, D, r, 16.0, 0.5, seed=6)


@pytest.mark.parametrize("B", [96, 1_100])
def test_dfeatures_over_features(B):
    """dfeatures written over the features: the bits of a call with a buffer of its own."""
    N, D, r = 20_000, 256, 0.2
    g = torch.Generator(device="cuda").manual_seed(3)
    X = torch.randn((B, D), generator=g, device="cuda")
    W = torch.randn((N, D), generator=g, device="cuda").mul_(0.01)
    labels = torch.randint(0, 40, (B,), generator=g, device="cuda")
    ctx = binding.Context(N, D, B, r, binding.PRECISION_BF16)
    cap = binding.pfc_num_sampled(N, B, r)
    idx = torch.zeros(cap, dtype=torch.int32, device="cuda")
    yl = torch.zeros(B, dtype=torch.int32, device="cuda")
    k = ctx.pfc_sample(labels, r, 1, 0, idx, yl)
    out = []
    for own in (True, False):
        feats = X.clone()
        dX = torch.zeros_like(X) if own else feats
        loss, dW = torch.zeros(1, device="cuda"), torch.zeros((cap, D), device="cuda")
        ctx.pfc_forward_backward(feats, W, idx, k, yl, 64.0, 0.5, loss, dX, dW)
        torch.cuda.synchronize()
        out.append((loss, dX, dW))
    for a, b in zip(*out):
        assert torch.equal(a, b)


@pytest.mark.parametrize("B,classes", [(1_024, 1), (1_024, 1_024), (1_023, 7), (3_000, 2), (3_000, 2_900)])
def test_first_sample_of_a_class(B, classes):
    """One label in the whole batch, as many labels as samples (the hash table of a window at its
    fullest), windows that share labels or hardly any."""
    N, D, r = 6_000, 256, 0.5
    rng = np.random.default_rng(7)
    X = rng.standard_normal((B, D)).astype(np.float32)
    W = (rng.standard_normal((N, D)) * 0.01).astype(np.float32)
    labels = rng.permutation(N)[np.arange(B) % classes]
    ctx = binding.Context(N, D, B, r, binding.PRECISION_FP32)
    idx, yl, k = gpu_sample(ctx, labels, r, 0, 0)
    idx = idx[:k]
    loss, dX, dWn = gpu_forward_backward(ctx, X, torch.from_numpy(W).cuda(), idx, yl, 16.0, 0.5)
    assert ctx.pfc_check() == binding.PFC_OK
    o = O.forward_backward(X, W[idx.astype(np.int64)], yl, 16.0, 0.5)
    tol = GRAD_TOL[binding.PRECISION_FP32]
    assert abs(loss - o["loss"]) <= LOSS_TOL[binding.PRECISION_FP32] * abs(o["loss"])
    assert rel_max(dX, o["dX"]) <= tol and rel_max(dWn, o["dWn"]) <= tol
