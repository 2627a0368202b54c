"""The library's host code against a HIP runtime in host memory (CPU only): what no machine with one
GPU and a healthy runtime can show.  The built library is linked behind tests/host/fake_hip.cpp, whose
functions take the place of the HIP runtime's; each case of tests/host/host_cases.cpp is one run."""
import os
import subprocess

import pytest

from paper_1810_08137_amd import ugks

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "host")
CLANG = "/opt/rocm/llvm/bin/clang++"

CASES = [
    "per_thread_stream",
    "other_device",
    "set_is_whole",
    "no_pinned_memory",
    "under_capture",
    "one_solver_at_a_time",
    "batch_workgroups",
    "static_scratch",
    "threads_that_do_not_start",
]


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("ROCm toolchain missing")
    exe = str(tmp_path_factory.mktemp("host") / "host_cases")
    r = subprocess.run(
        [CLANG, "-O1", "-g", "-std=c++17", "-pthread", "-rdynamic", "-D__HIP_PLATFORM_AMD__",
         "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"),
         "-I" + os.path.join(ROOT, "paper_1810_08137_amd", "csrc"),
         os.path.join(HERE, "fake_hip.cpp"), os.path.join(HERE, "host_cases.cpp"),
         ugks.LIB_PATH, "-Wl,-rpath," + os.path.dirname(ugks.LIB_PATH), "-o", exe],
        capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.mark.parametrize("case", CASES)
def test_host_code(program, case):
    r = subprocess.run([program, case], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
