"""Host rules of pfc_sample (csrc/pfc_sample_plan.h), compiled for the CPU: wherever the window
selection is chosen, its lists hold what falls into them, for everything the entry points accept."""
import ctypes
import math
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2203_15565_amd", "csrc")
FULL = 0xFFFFFFFF

_SRC = r"""
#include "pfc_sample_plan.h"
extern "C" int plan(int64_t N, int64_t crn, int64_t B, uint32_t mask, double* out) {
  const pfc::SelectWindow w = pfc::select_window(N, crn, B);
  out[0] = w.lo; out[1] = w.width; out[2] = w.shift; out[3] = w.expected;
  out[4] = pfc::window_bin_classes(N, w);
  out[5] = pfc::window_list_cap(N, B);
  out[6] = pfc::sample_cls_log2(N); out[7] = pfc::sample_blocks(N);
  out[8] = pfc::kBinList; out[9] = pfc::kLocalList; out[10] = pfc::kWindowBatch;
  out[11] = pfc::kWindowBins; out[12] = pfc::kMissClasses; out[13] = pfc::window_pos_cap(B);
  out[14] = pfc::sample_write_blocks(N); out[15] = pfc::sample_write_log2(N); out[16] = pfc::sample_count_cap(N);
  const int64_t scan = pfc::sample_write_blocks(N) << (pfc::sample_write_log2(N) - pfc::sample_cls_log2(N));
  out[17] = scan; out[18] = pfc::list_parts((int)scan); out[19] = pfc::kMaxClsLog2;
  return pfc::window_select(N, crn, B, mask, w) ? 1 : 0;
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    gxx = shutil.which("g++") or shutil.which("c++")
    if not gxx:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("plan")
    src, lib = d / "plan.cpp", d / "libplan.so"
    src.write_text(_SRC)
    subprocess.run([gxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(lib)],
                   check=True)
    f = ctypes.CDLL(str(lib)).plan
    f.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int64, ctypes.c_uint32,
                  ctypes.POINTER(ctypes.c_double)]
    keys = ("lo", "width", "shift", "expected", "bin", "list_cap", "cls_log2", "blocks", "bin_list",
            "local_list", "window_batch", "bins", "miss_classes", "pos_cap", "write_blocks", "write_log2", "count_cap",
            "scan", "parts", "max_log2")

    def call(N, crn, B, mask=FULL):
        out = (ctypes.c_double * len(keys))()
        taken = f(N, crn, B, mask, out)
        return bool(taken), dict(zip(keys, out))
    return call


def _forms(n):
    rng = random.Random(1)
    for _ in range(n):
        N = int(math.exp(rng.uniform(0.0, math.log(2**31 - 1))))
        B = int(math.exp(rng.uniform(0.0, math.log(2**20))))
        r = math.exp(rng.uniform(math.log(1e-9), 0.0))
        yield max(N, 1), max(1, min(N, math.ceil(r * N))), max(B, 1)
    for N in (2**20, 2**24, 20_971_520, 2**31 - 1):
        for B in (2**16, 2**17, 2**18, 2**20):
            yield N, N // 2, B
            yield N, max(1, N // 8), B


def test_window_lists_hold_what_falls_into_them(plan):
    taken = 0
    for N, crn, B in _forms(20_000):
        window, p = plan(N, crn, B)
        assert (int(p["width"]) >> int(p["shift"])) < p["bins"], (N, crn, B)
        assert p["blocks"] <= 640 or N > 20_971_520, (N, crn, B)
        if not window:
            continue
        taken += 1
        assert B <= p["pos_cap"] <= p["window_batch"]
        # the end bin, the list of one workgroup, the list of the call: 8 standard deviations
        assert p["bin"] + 8 * math.sqrt(p["bin"]) <= p["bin_list"], (N, crn, B)
        mean = p["expected"] / N * min(N, 2.0 ** p["cls_log2"])
        assert mean + 8 * math.sqrt(mean) <= p["local_list"], (N, crn, B)
        assert p["expected"] + 8 * math.sqrt(p["expected"]) <= p["list_cap"], (N, crn, B)
        # 6 standard deviations around every rank at which the selection can end
        for rank, edge in ((crn, p["lo"]), (max(0, crn - B), p["lo"] + p["width"] + 1)):
            q = rank / N
            sigma = math.sqrt(N * q * (1 - q))
            got = N * (1 - edge / 2**32)      # classes at or above that edge of the window
            if rank == crn:
                assert got >= min(N, crn + 6 * sigma) - 1e-3, (N, crn, B)
            else:
                assert got <= max(0.0, rank - 6 * sigma) + 1e-3, (N, crn, B)
    assert taken > 5_000


def test_parts_of_the_list_and_counts_hold_what_is_written(plan):
    """sample_scan leaves a count for each of its workgroups, whole ones of sample_write, and appends to one
    part of the list; a part that overflows costs a selection of every workgroup for itself."""
    sizes = [(N, max(1, N // d), B) for e in range(10, 15) for n in (63, 64, 65, 71, 512, 513, 639, 640)
             for N in ((n << e) - 1, n << e, (n << e) + 1) for d in (1, 2, 10) for B in (1, 64, 1_000, 65_536)]
    uneven = 0
    for N, crn, B in list(_forms(20_000)) + sizes:
        window, p = plan(N, crn, B)
        scan, parts, write = int(p["scan"]), int(p["parts"]), int(p["write_blocks"])
        assert p["cls_log2"] <= p["write_log2"] <= min(p["cls_log2"] + 1, p["max_log2"])
        # every class in a workgroup of either launch; counts within what the scratch has room for
        assert scan << int(p["cls_log2"]) >= N and write << int(p["write_log2"]) >= N, N
        assert p["blocks"] <= scan <= p["count_cap"] and write <= p["count_cap"], N
        assert write <= 512 or p["write_log2"] == p["max_log2"], N
        # a context whose largest call is this one, or any larger; parts of whole workgroups
        for B_max in (B, 2 * B, 2**20):
            cap = int(plan(N, crn, B_max)[1]["list_cap"]) // parts
            most = min(-(-scan // parts) * 2.0 ** p["cls_log2"], N) * p["expected"] / N
            if window:
                assert most + 8 * math.sqrt(most) <= cap, (N, crn, B, B_max)
        uneven += window and scan % parts != 0
    assert uneven > 1_000


def test_large_batches_and_moved_scores_take_the_radix_passes(plan):
    for N in (93_431, 2_059_906, 10_000_000, 2**24):
        assert plan(N, max(N // 10, 2048), 2048)[0]
        assert not plan(N, max(N // 10, min(N, 2**17)), 2**17)[0]
        assert not plan(N, N // 10, 512, 0x3FF)[0] and not plan(N, N // 10, 512, 0)[0]
    assert plan(9001, 1801, 40, 0x3FF)[0]                       # a miss costs little there
    assert plan(655_361, 6554, 300, 0xFFFFF000)[0]              # ties, but where the window is
    assert not plan(655_361, 6554, 300, 0xFFFF0000)[0]          # ten classes to a score: not any more
    assert plan(2_059_906, 1, 16_384)[0]                        # the classes of the batch alone


# (classes, ratio, samples): 512 .. 640 workgroups of sample_scan, half as many of sample_write, where the window took 60 to
# 80 % of the time of the radix passes; either side of the line, where the two were 10 % or more apart
@pytest.mark.parametrize("N,r,B,window", [
    (527_360, 0.1, 8_192, True), (1_187_840, 0.1, 8_192, True), (1_143_244, 0.5, 8_064, True), (2_390_744, 0.5, 7_615, True),
    (4_751_360, 0.1, 16_384, True), (8_437_760, 0.1, 16_384, True), (9_502_720, 0.1, 24_576, True),
    (93_431, 0.1, 8_192, True), (2_059_906, 1e-9, 65_536, True), (6_553_600, 0.1, 32_768, True),
    (527_360, 0.1, 24_576, False), (1_187_840, 0.1, 32_768, False), (2_109_440, 0.1, 49_152, False),
    (9_502_720, 0.1, 65_536, False), (90_000, 1.0, 32_768, False), (17_000_000, 0.01, 49_152, False)])
def test_the_way_that_was_measured_faster(plan, N, r, B, window):
    assert plan(N, max(1, math.ceil(r * N)), B)[0] is window
