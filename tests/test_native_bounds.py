"""Device functions of one block on the host, one thread per lane, under AddressSanitizer and
UndefinedBehaviorSanitizer (tests/native/host_lanes.h): every buffer in an allocation of its exact size,
buffer loads checked against both readings of the hardware's range check.  Host code only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_20917_amd", "csrc")
ROCM_INC = "/opt/rocm/include"

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(os.path.join(ROCM_INC, "hip")),
                                reason="needs g++ and the HIP headers")


def _run(tmp_path, name, *flags):
    exe = str(tmp_path / name)
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
           "-fno-omit-frame-pointer", "-w", "-D__HIP_PLATFORM_AMD__", *flags, "-I" + ROCM_INC, "-I" + CSRC,
           os.path.join(ROOT, "tests", "native", name + ".cpp"), "-o", exe, "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=900)
    assert r.returncode == 0, r.stderr[-4000:]
    # verify_asan_link_order=0: a library the environment preloads may come before the ASan runtime
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:verify_asan_link_order=0", UBSAN_OPTIONS="print_stacktrace=1")
    r = subprocess.run([exe], capture_output=True, text=True, timeout=900, env=env)
    assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-4000:])
    assert " 0 failures" in r.stdout


def test_staged_hexahedral_groups_stay_in_bounds(tmp_path):
    _run(tmp_path, "hex_staged_bounds")
