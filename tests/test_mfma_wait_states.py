"""A product written as inline assembly (at_mfma_acc) gets no wait states from the compiler: two must stand between the last
write of an operand and the product (what it puts before products it knows itself)."""
import os
import re
import shutil
import subprocess

import pytest

SOURCE = """
#include <hip/hip_runtime.h>
#include "attention_mfma.h"
using namespace varuna;
__global__ void probe(const float* a, float* out) {
  bf16x8 x, y;
  for (int i = 0; i < 8; ++i) { x[i] = (bf16)a[threadIdx.x * 8 + i]; y[i] = (bf16)a[512 + threadIdx.x * 8 + i]; }
  floatx16 c;
  for (int r = 0; r < 16; ++r) c[r] = 0.f;
  at_mfma_acc(c, x, y);
  at_mfma_settle();
  for (int r = 0; r < 16; ++r) out[threadIdx.x * 16 + r] = c[r];
}
"""


def test_wait_states_between_a_conversion_and_its_product(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2111_04007_amd", "csrc")
    (tmp_path / "probe.hip").write_text(SOURCE)
    subprocess.run([hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-I", csrc, "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-Wno-unknown-warning-option", "--cuda-device-only", "-S", str(tmp_path / "probe.hip"),
                    "-o", str(tmp_path / "probe.s")], check=True, capture_output=True)
    code = [line.split(";")[0].strip() for line in (tmp_path / "probe.s").read_text().splitlines()]
    code = [c for c in code if re.match(r"[vs]_\w+", c) or re.match(r"(global|ds|buffer|flat)_", c)]
    at = next(i for i, c in enumerate(code) if c.startswith("v_mfma"))
    states = 0
    for c in reversed(code[:at]):
        if c.startswith("v_cvt"):
            break
        states += int(c.split()[1], 0) + 1 if c.startswith("s_nop") else 1
    assert states >= 2, code[at - 6:at + 1]
