"""Builds the HIP shared library for gfx950 with hipcc (cross-compiles without a GPU)."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(HERE, "libvaruna_stage.so")
SOURCES = [  # compiled side by side
    os.path.join(HERE, "csrc", n) for n in ("gemm_fwd.hip", "gemm_dgrad.hip", "gemm_wgrad.hip", "gemm_f32.hip",
                                            "gemm_f32_bf16.hip", "attention.hip",
                                            "attention_edge.hip", "attention_f32.hip", "attention_f32_bf16.hip", "stage.hip")
]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unknown-warning-option",
]


def build(verbose: bool = True, extra_flags=()) -> str:
    """Compiles the sources side by side, then links them."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    with tempfile.TemporaryDirectory() as tmp:
        objs = [os.path.join(tmp, os.path.basename(s) + ".o") for s in SOURCES]

        def compile_one(src, obj):
            cmd = [hipcc, *HIPCC_FLAGS, *extra_flags, "-c", src, "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.run(cmd, check=True)

        with ThreadPoolExecutor(max_workers=len(SOURCES)) as pool:
            list(pool.map(compile_one, SOURCES, objs))
        subprocess.run([hipcc, "--offload-arch=gfx950", "-fPIC", "-shared", *objs, "-o", LIB_PATH], check=True)
    return LIB_PATH


if __name__ == "__main__":
    build(extra_flags=sys.argv[1:])
