"""The GEMM main loop with bf16 operands at its shortest reductions, for every size of tile: fewer slabs than it
holds in LDS, exactly as many, and the first counts at which buffers are used again."""
import pytest

from paper_2203_15565_amd import binding
from test_gpu_fused import test_fused_equals_two_calls as fused_equals_two_calls
from test_gpu_step import _fb_parity

pytestmark = pytest.mark.gpu

BF16 = binding.PRECISION_BF16


# logits: D / 64 slabs; dweight: as many as 64 samples go into the padded batch; dfeatures: slices of at least 4
@pytest.mark.parametrize("N,B,D", [(1_000, 100, D) for D in (64, 128, 192, 256, 320, 384)] +          # 64-tiles
                         [(10_000, 300, D) for D in (64, 128, 192, 256, 320, 384)] +                  # 128-tiles
                         [(16_384, 1_024, 320), (51_200, 256, 512), (20_000, 512, 448)])              # 256-tiles
def test_few_slabs(N, B, D):
    _fb_parity(BF16, N, B, D, 1.0, 64.0, 0.5, N + B + D)


# fused: slabs of 32 samples, four to eight of them; half-height tiles: of 64
@pytest.mark.parametrize("B", [48, 130, 256])
def test_few_slabs_fused(B):
    fused_equals_two_calls(36_000, B, 512, 1.0, BF16, 36_000, False)
