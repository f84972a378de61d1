"""bf16: E lies in panels of 8 classes x the padded batch.  Parity where a panel, a slab of either backward product or
the tile that writes them ends: every pair of tiles of the logits (64, 128, 256) and of the backward launch."""
import pytest

from paper_2203_15565_amd import binding
from test_gpu_step import _fb_parity

pytestmark = pytest.mark.gpu

BF16 = binding.PRECISION_BF16


# samples: either side of a half wavefront, of a tile and of the padding that the other product asks for; classes:
# one more and one less than an octet, a slab and a tile; tiles of the logits and of the backward launch
# (tests/test_step_plan.py holds the rules to them)
FORMS = [(263, 100, 64, 64, 64),
         (511, 97, 128, 64, 64),          # either end of the padding
         (1025, 160, 192, 64, 64),
         (4_001, 500, 512, 64, 128),
         (9_001, 129, 256, 128, 64),
         (16_383, 513, 320, 128, 128),    # samples one past a tile
         (20_479, 700, 512, 256, 256),
         (16_897, 1025, 512, 128, 256),   # 128-tiles write 1280 samples
         (33_000, 1000, 448, 128, 256),
         (30_215, 403, 320, 256, 128)]    # 256-tiles write 512 samples


@pytest.mark.parametrize("N,B,D,logits,backward", FORMS)
def test_parity(N, B, D, logits, backward):
    _fb_parity(BF16, N, B, D, 1.0, 64.0 if B > 200 else 20.0, 0.5, N + B + D)
