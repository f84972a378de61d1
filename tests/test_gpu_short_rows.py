"""Rows of at most 128 floats share a wavefront: several centers to one in the gather and in the update.  Numbers of
classes around what a wavefront and a workgroup hold; unsampled rows keep their bytes; a bad id is reported."""
import numpy as np
import pytest

from oracle import pfc_oracle as O
from paper_2203_15565_amd import binding
from pfc_harness import ROW_GRAD_TOL, gpu_forward_backward, rel_max, row_rel_err, row_rel_max

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("k", [1, 2, 7, 8, 9, 31, 33, 255, 256, 257, 1030])
def test_gather_and_update(D, k):
    import torch
    print("short rows", D, k, flush=True)
    rng = np.random.default_rng(100 * D + k)
    N, B = 1500, 9
    X = rng.standard_normal((B, D)).astype(np.float32)
    W = (rng.standard_normal((N, D)) * 0.01).astype(np.float32)
    v = (rng.standard_normal((N, D)) * 0.001).astype(np.float32)
    idx = np.sort(rng.choice(N, size=k, replace=False)).astype(np.int32)
    yl = rng.integers(0, k, size=B).astype(np.int32)
    ctx = binding.Context(N, D, B, 1.0, binding.PRECISION_FP32)
    Wd, vd = torch.from_numpy(W).cuda(), torch.from_numpy(v).cuda()
    loss, dX, dW = gpu_forward_backward(ctx, X, Wd, idx, yl, 64.0, 0.5)
    W64, v64 = W.astype(np.float64), v.astype(np.float64)
    o = O.forward_backward(X, W64[idx], yl, 64.0, 0.5)
    # (the bars of the fp32 parity tests; one class alone has no gradient)
    if k > 1:
        assert rel_max(dW, o["dWn"]) <= 2e-5
        assert row_rel_max(dW, o["dWn"])[0] <= ROW_GRAD_TOL[binding.PRECISION_FP32]
        assert rel_max(dX, o["dX"]) <= 2e-5
    g = rng.standard_normal((k, D)).astype(np.float32)
    ctx.pfc_update(Wd, vd, torch.from_numpy(idx).cuda(), k, torch.from_numpy(g).cuda(), 0.1, 0.9)
    torch.cuda.synchronize()
    ctx.check()
    nrm = np.linalg.norm(W64[idx], axis=1, keepdims=True)
    wn = W64[idx] / nrm
    O.update(W64, v64, idx, (g - (g * wn).sum(axis=1, keepdims=True) * wn) / nrm, 0.1, 0.9)
    W1, v1 = Wd.cpu().numpy(), vd.cpu().numpy()
    rest = np.setdiff1d(np.arange(N), idx)
    assert W1[rest].tobytes() == W[rest].tobytes() and v1[rest].tobytes() == v[rest].tobytes()
    assert rel_max(v1[idx], v64[idx]) < 1e-5   # 32-bit sums of 64 and 128 products
    assert row_rel_err(W1[idx], W64[idx], np.linalg.norm(W64[idx], axis=1)) < 1e-5
    ctx.close()


@pytest.mark.parametrize("D", [64, 128])
def test_bad_id_is_reported_and_its_neighbours_are_updated(D):
    import torch
    print("short rows, bad id", D, flush=True)
    N, k = 40, 6
    rng = np.random.default_rng(D)
    W = torch.from_numpy(rng.standard_normal((N, D)).astype(np.float32)).cuda()
    v, g = torch.zeros_like(W), torch.ones(k, D, device="cuda")
    ctx = binding.Context(N, D, 4, 1.0, binding.PRECISION_FP32)
    good = W.clone()
    ctx.pfc_update(good, v.clone(), torch.tensor([3, 4, 5, 6, 7, 8], dtype=torch.int32, device="cuda"), k, g, 0.1, 0.9)
    ctx.check()
    ctx.pfc_update(W, v, torch.tensor([3, 4, -1, N, 7, 8], dtype=torch.int32, device="cuda"), k, g, 0.1, 0.9)
    assert ctx.pfc_check() == binding.PFC_ELABEL
    for row in (3, 4, 7, 8):
        assert torch.equal(W[row], good[row])
    ctx.close()
