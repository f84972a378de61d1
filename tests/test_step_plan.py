"""Host rules of forward/backward (csrc/pfc_step_plan.h), compiled for the CPU: the scratch of a context
holds what every call of its range leaves there, and is no larger than it has to be."""
import ctypes
import heapq
import math
import os
import random
import shutil
import subprocess

import pytest

import test_gpu_backward_launch as backward_launch
import test_gpu_logits_slim as logits_slim
import test_gpu_octets as octets
import test_gpu_slab_counts as slab_counts
from test_gpu_sum_pieces import EQUAL, INDEPENDENT

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2203_15565_amd", "csrc")

_SRC = r"""
#include "pfc_step_plan.h"
using namespace pfc;
extern "C" void plan(int cu, int es, int D, int B, int64_t k, double* out) {
  const int64_t kp = round_up(k, kPadK);
  const TileSize f = logits_tiles(cu, es, B, kp, D), b = backward_tiles(cu, es, B, kp, D);
  const int Bp = (int)round_up(B, std::max<int>(f, b)), Dp = (int)round_up(D, b == TILES_256 ? 256 : kPadD);
  const BackwardShape s = backward_shape(cu, es, b, Bp, Dp, D, kp);
  out[0] = f; out[1] = b; out[2] = Bp; out[3] = Dp; out[4] = kp;
  out[5] = s.splits; out[6] = s.slabs_per; out[7] = s.dx.splits; out[8] = s.dx.slabs_per;
  out[9] = s.dx.wgs; out[10] = s.dx.tiles_i; out[11] = s.dx.tiles_d; out[12] = s.dx.slabs_total;
  out[13] = fits_one_kernel(cu, D, kp); out[14] = tile_bk(es); out[15] = s.dw_first;
  out[16] = es == 4 && f == TILES_64 && logits_slim(cu, B, kp);
}
extern "C" int64_t slabs(int64_t cu, int64_t na, int64_t a, int64_t nb, int64_t b) {
  return launch_slabs(cu, na, a, nb, b);
}
extern "C" void scratch(int cu, int D, int B_max, int64_t k_cap, double* out) {
  out[0] = (double)part_floats(cu, D, B_max);
  out[1] = (double)rowpart_floats(cu, B_max, round_up(k_cap, kPadK));
}
"""
_KEYS = ("logits", "backward", "Bp", "Dp", "kp", "dw_splits", "dw_slabs", "dx_splits", "dx_slabs", "dx_wgs",
         "tiles_i", "tiles_d", "dx_total", "one_kernel", "bk", "dw_first", "slim")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    gxx = shutil.which("g++") or shutil.which("c++")
    if not gxx:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("step_plan")
    src, out = d / "plan.cpp", d / "libplan.so"
    src.write_text(_SRC)
    subprocess.run([gxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(out)],
                   check=True)
    so = ctypes.CDLL(str(out))
    vp = ctypes.POINTER(ctypes.c_double)
    so.plan.argtypes = [ctypes.c_int] * 4 + [ctypes.c_int64, vp]
    so.slabs.argtypes, so.slabs.restype = [ctypes.c_int64] * 5, ctypes.c_int64
    so.scratch.argtypes = [ctypes.c_int] * 3 + [ctypes.c_int64, vp]
    return so


def _plan(lib, cu, es, D, B, k):
    out = (ctypes.c_double * len(_KEYS))()
    lib.plan(cu, es, D, B, k, out)
    return {n: int(v) for n, v in zip(_KEYS, out)}


def _scratch(lib, cu, D, B, k):
    out = (ctypes.c_double * 2)()
    lib.scratch(cu, D, B, k, out)
    return int(out[0]), int(out[1])


def _up(x, m):
    return -(-x // m) * m


def _log(rng, hi):
    return max(1, int(math.exp(rng.uniform(0.0, math.log(hi)))))


def _forms(n):
    """(compute units, bytes of an operand, D, largest batch, largest class set) and calls in that range"""
    rng = random.Random(2)
    for i in range(n):
        cu = 256 if i % 8 else rng.choice([64, 208, 304])
        es = rng.choice([2, 4])
        D = 64 * rng.randint(1, 16)
        B_max, k_cap = _log(rng, 2**20), _log(rng, 2**25 if es == 2 else 2**24)
        calls = [(B_max, k_cap), (1, k_cap), (B_max, 1), (_log(rng, B_max), k_cap), (B_max, _log(rng, k_cap)),
                 (_log(rng, B_max), _log(rng, k_cap))]
        yield cu, es, D, B_max, k_cap, calls


def test_scratch_holds_every_call(lib):
    tiles = set()
    for cu, es, D, B_max, k_cap, calls in _forms(20_000):
        parts, rows = _scratch(lib, cu, D, B_max, k_cap)
        for B, k in calls:
            p = _plan(lib, cu, es, D, B, k)
            form = (cu, es, D, B_max, k_cap, B, k, p)
            tiles.add((es, p["logits"], p["backward"]))
            front = p["dx_splits"] * p["Bp"] * p["Dp"]
            behind = p["dw_splits"] * p["kp"] * p["Dp"] if p["dw_splits"] > 1 else 0
            assert front + behind <= parts, form
            assert p["kp"] // p["logits"] * p["Bp"] <= rows, form
            # whole tiles, slices that cover the sums, none of them empty
            assert p["Bp"] % p["backward"] == 0 and p["Dp"] % p["backward"] == 0, form
            assert p["kp"] % p["backward"] == 0 and p["Bp"] >= B and p["Dp"] >= D, form
            assert (p["dx_splits"] - 1) * p["dx_slabs"] < p["dx_total"] <= p["dx_splits"] * p["dx_slabs"], form
            total = p["Bp"] // p["bk"]
            assert (p["dw_splits"] - 1) * p["dw_slabs"] < total <= p["dw_splits"] * p["dw_slabs"], form
            assert p["dx_wgs"] % 8 == 0 and p["dx_wgs"] >= p["tiles_i"] * p["tiles_d"] * p["dx_splits"], form
            if p["one_kernel"]:      # its dfeatures tiles are 128 or 256 wide, and dweight is in one piece
                assert p["backward"] >= 128 and p["dw_splits"] == 1, form
            # fp32: a 256-tile has no pieces, so only large batches that fill them take them, in short sums
            if es == 4 and p["backward"] == 256:
                assert p["Bp"] > 2048 and not p["one_kernel"], form
                assert 100 * p["Bp"] <= 105 * B and 100 * p["Dp"] <= 115 * _up(D, 128), form
                assert max(p["dw_slabs"], p["dx_slabs"]) * p["bk"] <= 4096, form
    assert len(tiles) >= 12


# (samples, classes, D, products of one uninterrupted fp32 sum of dweight and of dfeatures, at most): 256-tiles
# would end first by the estimate, but in sums of up to 4096; large batches whose 256-tiles could do with half
# as many slices
@pytest.mark.parametrize("B,k,D,dw,dx", [
    (4_096, 33_000, 64, 512, 256), (5_000, 20_000, 576, 512, 256), (3_864, 29_707, 1_024, 512, 256),
    (4_096, 8_000, 320, 512, 256), (2_500, 40_000, 256, 512, 256), (2_100, 3_000, 512, 512, 256),
    (2_048, 16_000, 512, 512, 256), (512, 9_344, 512, 512, 256),
    (4_774, 8_175, 256, 608, 640), (14_099, 2_330, 256, 512, 640), (11_951, 4_445, 256, 832, 928)])
def test_fp32_sums_stay_short(lib, B, k, D, dw, dx):
    p = _plan(lib, 256, 4, D, B, k)
    pieces = (512, 256) if p["backward"] < 256 and not p["one_kernel"] else (4096, 4096)
    assert min(p["dw_slabs"] * p["bk"], pieces[0]) <= dw, p
    assert min(p["dx_slabs"] * p["bk"], pieces[1]) <= dx, p


# (the GPU tests of these sums are about the tiles and slices that they name)
@pytest.mark.parametrize("B,k,D,tile,dw,dx", [c[:3] + c[5:] for c in EQUAL] + INDEPENDENT)
def test_sums_of_the_gpu_tests(lib, B, k, D, tile, dw, dx):
    p = _plan(lib, 256, 4, D, B, k)
    assert (p["backward"], p["dw_splits"], p["dx_splits"]) == (tile, dw, dx) and not p["one_kernel"]


def _bf16(lib, N, B, D, *keys):
    p = _plan(lib, 256, 2, D, B, N)
    return tuple(p[n] for n in keys)


# (likewise the forms that the GPU tests name: a rule that moves them leaves a kernel without its test)
def test_forms_of_the_gpu_tests(lib):
    for N, B, D, *form in backward_launch.BF16_FORMS:
        assert _bf16(lib, N, B, D, "logits", "backward", "dw_splits", "dx_splits") == tuple(form), (N, B, D)
    for N, B, D, logits, backward in octets.FORMS:
        assert _bf16(lib, N, B, D, "logits", "backward") == (logits, backward), (N, B, D)
    pairs = {f[3:5] for f in octets.FORMS}
    assert pairs == {(64, 64), (64, 128), (128, 64), (128, 128), (128, 256), (256, 128), (256, 256)}
    rng = random.Random(4)
    for _ in range(20_000):      # .. and no other pair is reached
        B, k, D = _log(rng, 2**16), _log(rng, 2**20), 64 * rng.randint(1, 16)
        assert _bf16(lib, k, B, D, "logits", "backward") in pairs, (B, k, D)
    for N, B, D, bf16, fp32 in slab_counts.FORMS:
        for es, form in ((2, bf16), (4, fp32)):
            p = _plan(lib, 256, es, D, B, N)
            assert (p["logits"], p["backward"]) == form, (es, N, B, D)
    # the last launch of one sample to a workgroup, and of four because of the batch
    for es in (2, 4):
        assert all(_plan(lib, 256, es, 192, B, 20_000)["dx_splits"] >= 12 for B in (256, 257))
        assert _plan(lib, 256, es, 1_024, 7, 40_000)["dx_splits"] >= 12
    assert all(_plan(lib, 256, 4, D, B, N)["slim"] for N, B, D in logits_slim.SLIM)
    for D in (64, 512, 832):     # the bits of slim tiles against those of 64-tiles
        assert [(_plan(lib, 256, 4, D, B, 8_192)["logits"], _plan(lib, 256, 4, D, B, 8_192)["slim"])
                for B in (64, 128)] == [(64, 1), (64, 0)]


def _ends_at(cu, p, es, dw_splits, dx_splits):
    """(slabs until the last compute unit is done, the mean over all of them) of a backward launch of
    256-tiles with these slices, the longer ones first, each workgroup with the edge of the rule's
    estimate, by simulation"""
    edge = 10 if es == 2 else 2
    dw_slabs, dx_slabs = -(-p["Bp"] // p["bk"] // dw_splits), -(-p["dx_total"] // dx_splits)
    dx = [dx_slabs + edge] * (p["tiles_i"] * p["tiles_d"] * dx_splits)
    dw = [dw_slabs + edge] * (p["kp"] // 256 * (p["Dp"] // 256) * dw_splits)
    free = [0] * cu
    for n in sorted(dw + dx, reverse=True):
        heapq.heapreplace(free, free[0] + n)
    return max(free), sum(free) / cu


# (operand bytes, D, samples, classes, and in bf16 the slices by number alone that made the launch 10 .. 25 %
# slower; fp32 operands had 128- and 64-tiles)
@pytest.mark.parametrize("es,D,B,k,before", [
    (2, 512, 4_096, 20_000, (1, 4)), (2, 512, 3_000, 20_000, (1, 5)), (2, 512, 8_192, 20_000, (1, 2)),
    (2, 1_024, 4_096, 20_000, (1, 2)), (4, 512, 16_384, 3_000, None), (4, 512, 8_192, 16_000, None),
    (4, 512, 8_192, 5_000, None), (4, 256, 32_768, 16_854, None), (4, 512, 65_536, 3_000, None),
    (4, 512, 4_096, 20_000, None)])
def test_large_batches_load_the_gpu_evenly(lib, es, D, B, k, before):
    p = _plan(lib, 256, es, D, B, k)
    assert p["backward"] == 256 and p["dw_first"] == (p["dw_slabs"] > p["dx_slabs"])
    end, mean = _ends_at(256, p, es, p["dw_splits"], p["dx_splits"])
    if before:
        assert end <= 0.9 * _ends_at(256, p, es, *before)[0], (end, p)
    else:
        assert end <= 1.16 * mean, (end, mean, p)


def test_estimate_of_a_launch_is_the_simulation(lib):
    rng = random.Random(7)
    for _ in range(3_000):
        cu = rng.choice([1, 3, 64, 256])
        a = rng.randint(1, 60)
        b = rng.randint(1, a)
        na, nb = rng.randint(0, 4 * cu), rng.randint(0, 4 * cu)
        if na == 0:
            continue
        free = [0] * cu
        for n in [a] * na + [b] * nb:
            heapq.heapreplace(free, free[0] + n)
        assert lib.slabs(cu, na, a, nb, b) == max(free), (cu, na, a, nb, b)


# (samples, classes, D, tiles of the backward launch): bf16 forms that 256-tiles made 4 - 8 % longer although the estimate
# has them 6 % and more shorter than 128-tiles, and forms that another size made 6 - 13 % shorter
@pytest.mark.parametrize("B,k,D,tile", [
    (187, 29_073, 576, 128), (138, 29_491, 640, 128), (237, 23_720, 832, 128), (474, 18_827, 896, 128),
    (414, 36_133, 448, 128), (531, 51_903, 448, 128), (484, 24_076, 768, 256),
    (1_296, 3_787, 896, 128), (1_105, 9_076, 576, 128), (1_952, 5_676, 448, 128), (1_891, 15_915, 448, 128),
    (931, 1_881, 1_024, 64), (921, 2_393, 512, 64), (170, 2_469, 128, 64)])
def test_bf16_backward_tiles(lib, B, k, D, tile):
    assert _plan(lib, 256, 2, D, B, k)["backward"] == tile


def test_scratch_stays_small(lib):
    """64 slices of the whole batch and two row sums for every 128 classes are what a context took before
    64-tiles and the saved label rows: what was accepted then has to fit now."""
    for cu, es, D, B_max, k_cap, _ in _forms(5_000):
        parts, rows = _scratch(lib, cu, D, B_max, k_cap)
        Bp, Dp, kp = _up(B_max, 256), _up(D, 256), _up(k_cap, 256)
        before = 64 * Bp * Dp + 2 * (kp // 128) * Bp
        assert parts + Bp * D + 2 * rows <= before + 2 * 2048 * cu + Bp * D * (Bp <= 4 * cu), (cu, D, B_max, k_cap)
    parts, rows = _scratch(lib, 256, 1024, 2**20, 2**20)
    assert 4 * parts <= 5 << 30 and 4 * rows <= 33 << 30
