"""The kernels' host side, compiled for the CPU alone with the HIP runtime replaced by stand-ins (tests/host_dispatch_driver.cpp): what a rule
promises the dispatcher, the launcher behind it takes, as built and with the build-time knobs that leave a kernel out."""
import os
import re
import subprocess

import pytest

from paper_2205_14756_amd import build as msla_build

SOURCES = ["k_project.hip", "k_apply.hip", "k_small.hip", "k_ffn.hip", "k_ffn_fused.hip"]


@pytest.mark.skipif(not os.path.exists(msla_build.HIPCC), reason="needs hipcc")
@pytest.mark.parametrize("knobs", [[], ["-DMSLA_APPLY_NO_WS"]], ids=["as_built", "without_the_weight_stationary_apply"])
def test_what_a_rule_promises_a_launcher_takes(tmp_path, knobs):
    objects = []
    for src in SOURCES:
        objects.append(str(tmp_path / (src + ".o")))
        subprocess.run([msla_build.HIPCC, "--offload-host-only", "-O0", "-std=c++17", "-w", *knobs, "-c", os.path.join(msla_build.CSRC, src), "-o", objects[-1]],
                       check=True, capture_output=True, timeout=300)
    # (the device code that the host side would register is not there)
    symbols = subprocess.run(["nm", *objects], check=True, capture_output=True, text=True, timeout=60).stdout
    device = sorted(set(re.findall(r"U (__hip_fatbin\w*)$", symbols, flags=re.M)))
    exe = str(tmp_path / "host_dispatch")
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-w",
                    os.path.join(os.path.dirname(os.path.abspath(__file__)), "host_dispatch_driver.cpp"), *objects, "-no-pie",
                    *[f"-Wl,--defsym,{d}=0" for d in device], "-o", exe], check=True, capture_output=True, timeout=300)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, (run.stdout + run.stderr)[-3000:]
    assert "host dispatch ok" in run.stdout
