"""The two backward products share one launch, and the size of the GEMM tiles follows from the
problem: parity where the launch changes its shape -- from one tile size to the next, from one slice
of the classes to several, with the batch cut into slices, with a last slice shorter than the
others, and with batches and rows that end inside a tile."""
import pytest

from paper_2203_15565_amd import binding
from test_gpu_step import _fb_parity

pytestmark = pytest.mark.gpu

# (N, B, D, r)
CASES = [
    (32_512, 64, 256, 1.0),     # 127 big tiles: small ones are taken
    (32_513, 64, 256, 1.0),     # 128 big tiles: big ones, last tile with one class
    (1_000, 64, 512, 0.256),    # one tile of 256 classes, one slice of dfeatures
    (1_000, 64, 512, 0.257),    # two of them, the second with one class
    (6_000, 1_024, 64, 0.5),    # batch of a whole number of tiles, D narrower than a tile
    (50_000, 2_049, 320, 1e-9),  # classes of the batch alone: batch cut into slices
    (50_000, 4_096, 256, 1e-9),  # likewise, whole tiles
    (300, 65, 64, 1.0),         # 64-tiles, second tile of the batch with one sample, half a column tile
    (16_384, 128, 128, 1.0),    # bf16: 128 tiles of 128 classes: 64-tiles for logits and backward
    (16_385, 129, 128, 1.0),    # one more of each: 128-tiles
    (3_300, 512, 384, 1.0),     # three column tiles of 128
    (16_000, 1_024, 320, 1.0),  # 256-tiles for the logits alone (0.98 of a round), rows of 384
    (16_000, 1_000, 512, 1.0),  # 256-tiles everywhere, batch ends inside a tile
    (9_000, 300, 640, 1.0),     # fp32: 64-tiles, bf16: 128-tiles; five column tiles
    (8_192, 256, 512, 1.0),     # fp32: exactly one 128-tile per compute unit
]


@pytest.mark.parametrize("N,B,D,r", CASES)
@pytest.mark.parametrize("precision", [binding.PRECISION_FP32, binding.PRECISION_BF16])
def test_backward_launch_edges(precision, N, B, D, r):
    _fb_parity(precision, N, B, D, r, 64.0, 0.5, seed=5)
