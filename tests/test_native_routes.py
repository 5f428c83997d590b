"""Kernel routes of the library, checked without a device.

tests/native/helm_map_routes.cpp is linked against libnir.so and run with every device hidden: a launch
that is let through ends in NIR_EHIP, one that is refused in NIR_EINVAL, and nothing runs.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2606_20917_amd")
ROCM = "/opt/rocm"


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(os.path.join(ROCM, "include", "hip")),
                    reason="needs g++ and the HIP headers")
def test_gathered_coefficients_reach_gathering_kernels_only(tmp_path):
    exe = str(tmp_path / "helm_map_routes")
    cmd = ["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROCM, "include"),
           "-I" + os.path.join(PKG, "csrc"), os.path.join(ROOT, "tests", "native", "helm_map_routes.cpp"), "-o", exe,
           os.path.join(PKG, "libnir.so"), "-L" + os.path.join(ROCM, "lib"), "-lamdhip64",
           "-Wl,-rpath," + os.path.join(ROCM, "lib"), "-Wl,-rpath," + PKG]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1", ROCR_VISIBLE_DEVICES="")
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300, env=env)
    assert r.returncode == 0, (r.stdout[-4000:], r.stderr[-2000:])
    assert "0 failures" in r.stdout
