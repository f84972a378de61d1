"""The two backward products share one launch: parity where its shape changes -- from small to big
tiles, from one slice of the classes to several, with the batch cut into slices, with a last slice
shorter than the others."""
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
]


@pytest.mark.parametrize("N,B,D,r", CASES)
@pytest.mark.parametrize("precision", [binding.PRECISION_FP32, binding.PRECISION_BF16])
def test_backward_launch_edges(precision, N, B, D, r):
    _fb_parity(precision, N, B, D, r, 64.0, 0.5, seed=5)
