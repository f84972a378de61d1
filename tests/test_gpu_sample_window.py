"""pfc_sample at the edges of its two-launch select: number of workgroups, classes per workgroup, list
entries kept in registers, windows that hold everything, windows that miss, ties inside the window."""
import sys

import numpy as np
import pytest

from oracle import pfc_oracle as O
from paper_2203_15565_amd import binding
from pfc_harness import gpu_sample

pytestmark = pytest.mark.gpu


# N: one class, one bitmap word, one workgroup (1024 classes) and its neighbours; 63, 64 and 65
# workgroups; 640 workgroups of 1024 classes and one class more (2048 each).
# Entries of the window's list that each of 512 threads keeps in registers, by the list's expected length:
# 2 (655,360 classes: 669), 6 (655,361 at 0.01: 1,415), 16 (9,000: 3,392; 655,361 at 0.7: 5,204), 24 (300,001:
# 11,841); with 2,000,003 classes it is longer than 24 x 512 (17,520) and the rest is read again.
# Masks: 0xFFFFF000 leaves ties inside the window, 0x3FF makes every window miss (up to 10,240 classes; larger
# sets take the radix passes, see test_gpu_sample_routes.py).
@pytest.mark.parametrize("N,B,r,mask", [
    (1, 1, 1.0, None), (31, 9, 0.3, None), (33, 40, 1.0, None), (1023, 50, 0.99, None),
    (1024, 1024, 0.5, None), (1025, 3, 0.001, None), (9000, 3000, 1.0, None),
    (9000, 3000, 0.34, None), (64_512, 700, 0.2, None), (65_536, 700, 0.2, None),
    (65_537, 700, 0.2, 0xFFFFF000), (655_360, 300, 0.001, None), (655_361, 300, 0.7, None),
    (655_361, 300, 0.01, 0xFFFFF000), (70_001, 200, 0.3, 0x3FF), (3_000_001, 5000, 1e-9, None),
    (10_001, 700, 0.3, 0x3FF), (300_001, 9000, 0.2, None), (2_000_003, 12_000, 0.1, None)])
def test_sample_window_edges(N, B, r, mask):
    ctx = binding.Context(N, 64, B, r, binding.PRECISION_FP32)
    rng = np.random.default_rng(N + B)
    for step in range(3):       # calls in a row use the two sets of counters in turn
        b = B if step != 1 else max(1, B // 3)
        labels = rng.integers(0, N, size=b)
        if step == 2:
            labels[: b // 2] = labels[0]
        print("sample window", N, b, r, step, flush=True)
        sys.stdout.flush()
        idx, yl, k = gpu_sample(ctx, labels, r, 77, step, score_mask=mask)
        oidx, oyl, ok = O.sample(labels, N, r, 77, step,
                                 score_mask=0xFFFFFFFF if mask is None else mask)
        assert k == ok
        assert np.array_equal(idx[:k], oidx) and (idx[k:] == -7).all()
        assert np.array_equal(yl, oyl)
    assert ctx.pfc_check() == binding.PFC_OK
    ctx.close()
