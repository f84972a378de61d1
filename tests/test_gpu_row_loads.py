"""pfc_update by each way of loading W and v (row_policy: resident, reused, streamed): the same update of the sampled
rows, and no other row touched.  And the rule itself, which gather and update have to share."""
import ctypes
import os
import subprocess

import pytest

from paper_2203_15565_amd import binding, build

# N, D, B_max, k, which way
CASES = [(3_000, 64, 64, 700, 0), (3_000, 128, 64, 701, 0), (2_000, 1024, 64, 333, 0),
         (400_000, 64, 64, 2_001, 1), (200_000, 128, 64, 999, 1), (100_000, 256, 64, 501, 1), (80_000, 320, 64, 500, 1),
         (40_000, 640, 64, 77, 1), (30_000, 1024, 64, 130, 1),
         (400_000, 64, 4096, 33_001, 2), (200_000, 128, 4096, 31_001, 2), (80_000, 320, 4096, 26_001, 2)]


def test_the_rule(tmp_path):
    src, lib = tmp_path / "rule.cpp", tmp_path / "rule.so"
    src.write_text('#include "pfc_step_plan.h"\nextern "C" int rule(int es, long N, int D, int B, long k) {\n'
                   '  const pfc::RowPolicy p = pfc::row_policy(es, N, D, B, k);\n  return p.loads * 2 + p.gather_plain; }\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(os.path.dirname(build.__file__), "csrc"),
                    str(src), "-o", str(lib)], check=True)
    rule = ctypes.CDLL(str(lib)).rule
    rule.argtypes = [ctypes.c_int, ctypes.c_long, ctypes.c_int, ctypes.c_int, ctypes.c_long]
    for N, D, B, k, way in CASES:
        assert rule(2, N, D, B, k) >> 1 == way, (N, D, B, k)
    assert rule(2, 40_000, 512, 512, 40_000) == 0                # W and v stay, the rest does not fit beside them
    assert rule(2, 2_059_906, 512, 1024, 205_991) == 4
    # reused means that the gather keeps the rows
    assert all(rule(es, N, 512, B, N // 10) in (0, 1, 3, 4) for es in (2, 4) for N in (10_000, 90_000, 400_000, 9_000_000)
               for B in (1, 512, 16_384))
    # behind other data a plain gather was up to 9 % slower in steps of 107 MB and more, no slower up to 91
    assert rule(2, 40_000, 512, 512, 16_000) == 0 and rule(2, 45_000, 512, 256, 20_000) == 0
    assert rule(2, 300_000, 512, 512, 18_000) == 4 and rule(2, 700_000, 256, 128, 70_000) == 4
    assert rule(2, 350_000, 512, 256, 35_000) == 4 and rule(4, 300_000, 512, 512, 18_000) == 4
    assert rule(2, 90_000, 256, 1024, 18_000) == 1 and rule(2, 85_742, 128, 256, 25_724) == 1
    # .. but for rows of 64, where it was faster or even up to 207
    assert rule(2, 1_500_000, 64, 100, 150_000) == 3 and rule(2, 2_000_000, 64, 64, 200_000) == 3
    assert rule(2, 800_000, 64, 900, 80_000) == 3 and rule(2, 200_000, 64, 100, 200_000) == 1
    assert rule(2, 93_431, 512, 512, 9_344) == 3 and rule(4, 93_431, 512, 512, 9_344) == 3


@pytest.mark.gpu
@pytest.mark.parametrize("N,D,B,k,way", CASES)
def test_update(N, D, B, k, way):
    import torch
    print("update", N, D, B, k, way, flush=True)
    g = torch.Generator(device="cuda").manual_seed(N + D)
    W = torch.randn((N, D), generator=g, device="cuda") * 0.01
    v = torch.randn((N, D), generator=g, device="cuda")
    dW = torch.randn((k, D), generator=g, device="cuda") * 0.01
    idx = torch.randperm(N, generator=g, device="cuda")[:k].sort().values
    W0, v0 = W.clone(), v.clone()
    ctx = binding.Context(N, D, B, max(k / N, 1e-9), binding.PRECISION_BF16)
    lr, mu = 0.1, 0.9
    ctx.pfc_update(W, v, idx.int(), k, dW, lr, mu)
    assert ctx.pfc_check() == binding.PFC_OK
    ctx.close()
    w, p, d = W0[idx].double(), v0[idx].double(), dW.double()
    rn = 1.0 / w.norm(dim=1, keepdim=True)
    t = (d * w).sum(1, keepdim=True) * rn * rn
    vn = mu * p + (d - t * w) * rn
    wn = w - lr * vn
    # roundings of sums of D terms in trees (64 lanes of 4 .. 16) and of a few products: below 16 ulp of the terms
    terms = mu * p.abs() + (d.abs() + (d * w).abs().sum(1, keepdim=True) * rn * rn * w.abs()) * rn
    assert ((v[idx].double() - vn).abs() <= 16 * 2.0 ** -24 * terms).all()
    assert ((W[idx].double() - wn).abs() <= 16 * 2.0 ** -24 * (w.abs() + lr * terms)).all()
    W[idx], v[idx] = W0[idx], v0[idx]
    assert torch.equal(W, W0) and torch.equal(v, v0)
