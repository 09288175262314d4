"""Wait states ahead of lane writes in inline assembly: a vector instruction that
writes a scalar register needs two before another reads it, and the compiler does
not insert them in front of inline assembly (compiled for gfx950, looked at on
the CPU)."""

import os
import re
import subprocess

import pytest

from paper_2407_20731_amd import build as B

SRC = """
#include "isr.h"
#include "isr_common.cuh"
namespace isr {
extern "C" __global__ void k(u64* o, const double* x, double t) {
  const u64 b = ballot(x[threadIdx.x] >= t);
  u64 v = writelane64<0>(b, 0ull);
  v = writelane64<1>(bcast64(o[threadIdx.x], 5), v);
  o[threadIdx.x] = v;
}
}
"""


def _scalars(operand):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if m:
        return {f"s{k}" for k in range(int(m[1]), int(m[2]) + 1)}
    return {"vcc_lo", "vcc_hi"} if operand == "vcc" else {operand} if re.fullmatch(r"s\d+|vcc_(lo|hi)", operand) else set()


def test_two_wait_states_before_a_lane_write(tmp_path):
    try:
        hipcc = B.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not available")
    src, out = tmp_path / "k.hip", tmp_path / "k.s"
    src.write_text(SRC)
    flags = [f for f in B.COMMON + B.HIP_FLAGS if f != "-fPIC"]
    subprocess.run([hipcc, *flags, "-S", "--cuda-device-only", str(src), "-o", str(out)], check=True, capture_output=True)
    code = [re.split(r"[,\s]+", line.split(";")[0].strip()) for line in out.read_text().splitlines()]
    code = [c for c in code if re.match(r"[svdgb]\w*_", c[0])]
    writes = [i for i, c in enumerate(code) if c[0].startswith("v_writelane")]
    assert len(writes) == 4
    for i in writes:
        read, waited = _scalars(code[i][2]), 0
        for c in reversed(code[:i]):
            if c[0].startswith("v_") and _scalars(c[1]) & read:
                assert waited >= 2, (c, code[i])
                break
            waited += int(c[1]) + 1 if c[0] == "s_nop" else 1
