"""The loads from global memory to LDS are inline assembly, where the compiler inserts no wait states: in its output
for the GEMM main loops, an SGPR that the vector ALU has written must be five wait states old when such a load takes
its address from it (or the load takes a scalar copy), and M0 one."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2203_15565_amd import build

_SRC = r"""
#include "pfc_gemm.h"
using namespace pfc;
// tile indices from a division, as in the product's kernels
template <class Cfg>
__global__ __launch_bounds__(Cfg::THREADS) void tile(const __bf16* A, const __bf16* B, int64_t lda, int64_t ldb, int n,
                                                     int inner, float* C) {
  extern __shared__ __align__(16) char smem[];
  const int o = blockIdx.x / inner, i = blockIdx.x % inner;
  f32x16 acc[Cfg::TM][Cfg::TN];
  zero_acc<Cfg>(acc);
  gemm_tile<Cfg>(A + o * lda, lda, B + i * ldb, ldb, n, smem, acc);
  for (int a = 0; a < Cfg::TM; ++a)
    for (int b = 0; b < Cfg::TN; ++b)
      for (int r = 0; r < 16; ++r)
        C[((blockIdx.x * Cfg::THREADS + threadIdx.x) * Cfg::TM * Cfg::TN + a * Cfg::TN + b) * 16 + r] = acc[a][b][r];
}
#define TILE(...) template __global__ void tile<TileCfg<__bf16, __VA_ARGS__>>(const __bf16*, const __bf16*, int64_t, \
                                                                              int64_t, int, int, float*);
TILE(256, 256, 2, 4, false, false)
TILE(256, 256, 2, 4, true, true)
TILE(128, 128, 2, 4, false, true)
TILE(64, 64, 2, 2, true, true)
TILE(128, 512, 2, 4, true, true, 64, 4, 4)
"""


def _sgprs(op):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]|s(\d+)", op)
    if not m:
        return set()
    return {int(m[3])} if m[3] else set(range(int(m[1]), int(m[2]) + 1))


def _states(text):
    """(wait states since the vector ALU last wrote the address, since M0 was written, whether the address is a scalar
    copy of what the vector ALU has written) for every load to LDS; None where the instructions in front have no
    such write"""
    out, before = [], []
    for line in text.splitlines():
        line = line.split(";")[0].strip()
        if not line or line.startswith((".", "#")) or line.endswith(":"):
            continue
        name, _, rest = line.partition(" ") if " " in line else line.partition("\t")
        ops = [o.strip() for o in rest.split(",")]
        if name.startswith("global_load_lds"):
            regs, states, valu, m0, source, copied = _sgprs(ops[1]), 0, None, None, set(), False
            for n, o in reversed(before[-64:]):
                hit = _sgprs(o[0]) & regs
                if hit and n.startswith("v_") and valu is None:
                    valu = states
                copied = copied or (n.startswith("v_") and bool(_sgprs(o[0]) & source))
                if n.startswith("s_") and n != "s_nop":
                    regs, source = regs - hit, source - _sgprs(o[0])
                    if n == "s_mov_b64" and hit:
                        source = source | _sgprs(o[1])
                    if o[0] == "m0" and m0 is None:
                        m0 = states
                states += int(o[0], 0) + 1 if n == "s_nop" else 1
            out.append((valu, m0, copied))
        before.append((name, ops))
    return out


def test_the_states_are_counted():
    text = "v_readfirstlane_b32 s5, v1\ns_mov_b32 m0, s9\ns_nop 0\nglobal_load_lds_dwordx4 v2, s[4:5]\n"
    assert _states(text) == [(2, 1, False)]
    assert _states(text.replace("s_nop 0", "s_nop 4")) == [(6, 5, False)]
    assert _states("s_add_u32 s4, s4, s6\n" + text.replace("s5, v1", "s7, v1")) == [(None, 1, False)]
    copy = text.replace("s_nop 0", "s_mov_b64 s[2:3], s[4:5]").replace("v2, s[4:5]", "v2, s[2:3]")
    assert _states(copy) == [(None, 1, True)]


def test_wait_states_of_loads_to_lds(tmp_path):
    hipcc = build._hipcc()
    if not shutil.which(hipcc):
        pytest.skip("no hipcc")
    src, out = tmp_path / "tile.hip", tmp_path / "tile.s"
    src.write_text(_SRC)
    subprocess.run([hipcc, *build.HIPCC_FLAGS, "--cuda-device-only", "-S", str(src), "-o", str(out)], check=True,
                   stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    loads = _states(out.read_text())
    assert len(loads) > 100
    assert any(copied or valu is not None for valu, _, copied in loads)     # the case is there
    assert all(valu is None or valu >= 5 for valu, _, _ in loads)
    assert all(m0 is not None and m0 >= 1 for _, m0, _ in loads)
