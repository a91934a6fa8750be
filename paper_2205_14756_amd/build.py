"""Builds libmsla.so (the gfx950 kernels + the C ABI of include/msla.h) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmsla.so")
OBJ_DIR = os.path.join(HERE, "_build")

SOURCES = ["k_project.hip", "k_aggregate.hip", "k_aggregate_mfma.hip", "k_aggregate_small.hip", "k_aggregate32.hip", "k_apply.hip", "k_small.hip", "k_ffn.hip", "k_ffn_fused.hip", "k_softmax.hip", "k_backward.hip", "k_generic.hip", "k_layout.hip", "msla_static.hip", "msla_api.cpp"]
HEADERS = ["msla_device.h", "aggregate_sweep.h", "gemm_tile.h", "msla_kernels.h", os.path.join("..", "..", "include", "msla.h")]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# packed-fp32 code generation is switched off for every device compile
DEVICE_FLAGS = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function"]
# kernels whose MFMA results are consumed by vector instructions right away: let the matrix
# instructions write VGPRs instead of AGPRs (saves one copy per result register)
PER_SOURCE = {"k_aggregate_mfma.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
              "k_aggregate_small.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
              "k_aggregate.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
              "k_aggregate32.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"]}


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC] + COMMON + (DEVICE_FLAGS if src.endswith(".hip") else []) + PER_SOURCE.get(src, []) + \
          ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines() if "not a recognized feature" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{out}")
    if out.strip():
        sys.stderr.write(out + "\n")
    return obj


def is_stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    deps = [os.path.join(CSRC, s) for s in SOURCES + HEADERS]
    return any(os.path.getmtime(d) > t for d in deps)


def build(force: bool = True) -> str:
    if not force and not is_stale():
        return LIB
    os.makedirs(OBJ_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=4) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + f".tmp{os.getpid()}"
    r = subprocess.run([HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", tmp] + objs,
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(True))
