"""row_sums of equal values: its assembly writes a register before it has read all of its inputs, so
that the compiler must not give an input the register of an output, even where both start with the
same value. Compiles such a call for the GPU and follows the masked DPP adds of the listing on the
CPU: of ones, every lane holds the number of lanes that were added up."""
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

from paper_2412_12734_amd import build

SOURCE = """
#include "device_util.h"
extern "C" __global__ void sums(const float* in, float* out) {
  const float x = in[threadIdx.x];
  float v[%d];
  for (float& y : v) y = x;
  out[threadIdx.x] = gbb::row_sums(v);
}
"""
LANE = np.arange(16)
MOVES = {"row_mirror": 15 - LANE, "row_half_mirror": (LANE & 8) | (7 - (LANE & 7))}


@pytest.mark.parametrize("K", [3, 6, 12])
def test_equal_values_do_not_share_an_outputs_register(tmp_path, K):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    src, lst = tmp_path / "sums.hip", tmp_path / "sums.s"
    src.write_text(SOURCE % K)
    flags = [f for f in build.HIP_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([hipcc, *flags, "--cuda-device-only", "-S", "-I", build.CSRC, str(src), "-o",
                    str(lst)], check=True, stderr=subprocess.DEVNULL, cwd=os.path.dirname(src))
    regs = {}
    adds = 0
    for line in lst.read_text().splitlines():
        m = re.match(r"\s+v_add_f32_dpp (v\d+), (v\d+), (v\d+) (row_mirror|row_half_mirror) "
                     r"row_mask:0xf bank_mask:0x(\w)$", line)
        if not m:
            continue
        dst, a, b, move, mask = m.groups()
        val = lambda r: regs.setdefault(r, np.ones(16))
        on = (int(mask, 16) >> (LANE >> 2) & 1).astype(bool)
        regs[dst] = np.where(on, val(a)[MOVES[move]] + val(b), val(dst))
        adds += 1
    assert adds == {3: 4, 6: 8, 12: 18}[K]
    # inputs stay, the first fold adds two lanes, the second four (of K = 3's third value, which is
    # folded only here, two)
    fine = [np.full(16, n) for n in (1, 2, 4)]
    fine += [np.where(LANE & 4, 2, 4)] if K == 3 else []
    for r, v in regs.items():
        assert any(np.array_equal(v, f) for f in fine), (r, v)
