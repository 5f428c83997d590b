"""Device functions of one block on the host, one thread per lane, under AddressSanitizer,
UndefinedBehaviorSanitizer or ThreadSanitizer (tests/native/host_lanes.h): every buffer in an allocation
of its exact size, buffer loads checked against both readings of the hardware's range check, and no two
lanes at one value without a barrier between.  Host code only."""
import concurrent.futures as cf
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_20917_amd", "csrc")
ROCM_INC = "/opt/rocm/include"

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(os.path.join(ROCM_INC, "hip")),
                                reason="needs g++ and the HIP headers")


SANITIZERS = "address,undefined"


def _run(tmp_path, name, sanitize=SANITIZERS, sources=(), flags=("-O1", "-g")):
    exe = str(tmp_path / (name + "_".join(("", *flags, sanitize)).replace(",", "_")))
    cmd = ["g++", "-std=c++17", "-fsanitize=" + sanitize, "-fno-sanitize-recover=all", "-fno-omit-frame-pointer", "-w",
           "-D__HIP_PLATFORM_AMD__", *flags, "-I" + ROCM_INC, "-I" + CSRC,
           os.path.join(ROOT, "tests", "native", name + ".cpp"), *sources, "-o", exe, "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=900)
    assert r.returncode == 0, r.stderr[-4000:]
    # verify_asan_link_order=0: a library the environment preloads may come before the ASan runtime
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:verify_asan_link_order=0", UBSAN_OPTIONS="print_stacktrace=1")
    r = subprocess.run([exe], capture_output=True, text=True, timeout=900, env=env)
    assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-4000:])
    assert " 0 failures" in r.stdout


def _thread_sanitizer_runs(tmp_path):
    """Whether a program under ThreadSanitizer starts here (it needs a memory layout that some kernels'
    address randomisation does not give)."""
    src, exe = tmp_path / "probe.cpp", str(tmp_path / "probe")
    src.write_text("int main() { return 0; }\n")
    built = subprocess.run(["g++", "-fsanitize=thread", str(src), "-o", exe], capture_output=True, timeout=120)
    return built.returncode == 0 and subprocess.run([exe], capture_output=True, timeout=60).returncode == 0


def test_half_conversion_rounds_to_nearest_even(tmp_path):
    _run(tmp_path, "half_bits", flags=("-O2",))


def test_staged_hexahedral_groups_stay_in_bounds(tmp_path):
    _run(tmp_path, "hex_staged_bounds")


@pytest.mark.parametrize("shape", [1, 2, 3], ids=["prism", "tet", "pyr"])
def test_collapsed_groups_stay_in_bounds(shape, tmp_path):
    """Every order under AddressSanitizer, two of them under ThreadSanitizer where it runs."""
    sources = [os.path.join(CSRC, f) for f in ("api.cpp", "tables.cpp")]

    def one(job):
        P, sanitize = job
        # api.cpp makes the tables; the launches that it refers to are not linked in and not called
        flags = ("-O0", "-fpermissive", "-Wl,--unresolved-symbols=ignore-all", f"-DCHECK_SHAPE={shape}",
                 f"-DCHECK_PMIN={P}", f"-DCHECK_PMAX={P}")
        _run(tmp_path, "col_bounds", sanitize, sources, flags)

    threads = _thread_sanitizer_runs(tmp_path)
    jobs = [(P, "address") for P in range(10, 1, -1)] + [(P, "thread") for P in (6, 3) if threads]
    with cf.ThreadPoolExecutor(min(8, os.cpu_count() or 1)) as ex:
        list(ex.map(one, jobs))


def test_chain_factors_of_collapsed_points(tmp_path):
    _run(tmp_path, "col_chain", sources=[os.path.join(CSRC, "tables.cpp")])


def test_rows_at_the_end_of_the_index_range(tmp_path):
    _run(tmp_path, "row_sum_edges")
