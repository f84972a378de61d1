"""Device memory that a context takes."""
import pytest
import torch

from paper_2203_15565_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,D,B", [(4_096, 1_024, 65_536), (400_000, 64, 16_384)])
def test_context_takes_what_its_operands_need(N, D, B):
    """Operands, E and the caller-sized buffers; the partial sums of the backward launch are bounded by
    the GPU's size (64 slices of the batch would be 17 GB in the first case)."""
    print("context", N, D, B, flush=True)
    k = binding.pfc_num_sampled(N, B, 1.0)
    kp, Dp = -(-k // 256) * 256, -(-D // 256) * 256
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    before, _ = torch.cuda.mem_get_info()
    ctx = binding.Context(N, D, B, 1.0, binding.PRECISION_BF16)
    after, _ = torch.cuda.mem_get_info()
    ctx.close()
    need = 2 * (2 * B * Dp + kp * Dp + B * kp)            # Xn, Xs, Wn, E
    need += 4 * (3 * B * Dp + k * D + 2 * kp // 128 * B)  # one slice, label rows, label part; dWn; row sums
    assert before - after <= need + (512 << 20), (before - after, need)
