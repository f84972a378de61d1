"""pfc_sample where sample_scan and sample_write change form: one marking workgroup (512 labels) or several, two or
four labels to a thread (1024), the list in one part or eight (64 workgroups), one or two workgroups of sample_scan
to one of sample_write (512)."""
import numpy as np
import pytest

from oracle import pfc_oracle as O
from paper_2203_15565_amd import binding
from pfc_harness import gpu_sample

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [512, 513, 1024, 1025, 2049])
@pytest.mark.parametrize("N,r", [(64_513, 0.05), (524_288, 0.01), (524_289, 0.3), (655_300, 1e-9)])
def test_parts_of_the_sampler(N, B, r):
    ctx = binding.Context(N, 64, B, max(r, 0.01), binding.PRECISION_BF16)
    rng = np.random.default_rng(N + B)
    # spread out; every second class of a few words and the last ones; one class; spread out again
    draws = (lambda: rng.integers(0, N, B), lambda: np.where(rng.random(B) < 0.5, 2 * rng.integers(0, 300, B),
                                                             N - 1 - rng.integers(0, 70, B)),
             lambda: np.full(B, N - 1), lambda: rng.integers(0, N, B))
    for step, draw in enumerate(draws):
        labels = draw()
        print("sample parts", N, B, r, step, flush=True)
        idx, yl, k = gpu_sample(ctx, labels, r, 11, step)
        oidx, oyl, ok = O.sample(labels, N, r, 11, step)
        assert k == ok and np.array_equal(idx[:k], oidx) and np.array_equal(yl, oyl)
    assert ctx.pfc_check() == binding.PFC_OK
    ctx.close()
