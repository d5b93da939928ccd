"""Host checks in front of the fused launches (no GPU needed: every call is
refused before it would reach one)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2208_02427_amd")


def test_fused_pass_without_one_of_its_arrays_is_refused(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if shutil.which(hipcc) is None or not os.path.exists(os.path.join(PKG, "liblap.so")):
        pytest.skip("needs hipcc and a built liblap.so")
    exe = str(tmp_path / "fused_arguments")
    subprocess.run([hipcc, "--offload-host-only", "-std=c++17", "-O0", "-w", "-x", "hip",
                    os.path.join(ROOT, "tests", "native", "fused_arguments.cpp"), "-I", os.path.join(PKG, "csrc"),
                    "-x", "none", os.path.join(PKG, "liblap.so"), f"-Wl,-rpath,{PKG}", "-o", exe], check=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, run.stdout + run.stderr
