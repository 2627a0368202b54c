"""The library's host code against a HIP runtime in host memory (CPU only): what no machine with one
GPU and a healthy runtime can show.  The built library is linked behind tests/host/fake_hip.cpp, whose
functions take the place of the HIP runtime's; each case of tests/host/host_cases.cpp is one run."""
import os
import subprocess

import pytest

from paper_1810_08137_amd import ugks
from tests import test_gpu_face_chunks as FACES
from tests import test_gpu_update_nodes as NODES
from tests import test_gpu_update_nodes_more as MORE

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
    "threads_share_the_pool",
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


def _kernels(program, nx, ny, nu, nv, precision="fp64", dof=0, prandtl=1.0, bc=1):
    """Names of the kernels that one step of such a solver launches."""
    r = subprocess.run([program, "kernels"] + [str(x) for x in (
        nx, ny, nu, nv, int(precision == "fp32_store"), dof, prandtl, bc)],
        capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


# Solvers whose step is faster by node (or by line) by more than 2%, as measured (us by node, by line),
# those of tests/test_gpu_update_nodes.py (all but one split) and of
# tests/test_gpu_update_nodes_more.py.
MEASURED = [
    (dict(nx=80, ny=40, nu=49, nv=49), True),                              # 88.1, 92.3
    (dict(nx=200, ny=50, nu=101, nv=101), True),                           # 911, 938
    (dict(nx=120, ny=60, nu=49, nv=49), True),                             # 158.7, 164.4
    (dict(nx=120, ny=60, nu=29, nv=29, precision="fp32_store"), True),     # 61.3, 64.0
    (dict(nx=278, ny=40, nu=67, nv=49, precision="fp32_store"), True),     # 194.8, 204.1
    (dict(nx=71, ny=80, nu=64, nv=51, precision="fp32_store"), True),      # 131.6, 135.5
    (dict(nx=92, ny=97, nu=24, nv=61, precision="fp32_store"), True),      # 94.3, 109.9
    (dict(nx=77, ny=36, nu=67, nv=65), False),                             # 126.0, 122.8
    (dict(nx=188, ny=12, nu=60, nv=65), False),                            # 85.8, 83.4
    (dict(nx=94, ny=44, nu=71, nv=8, dof=1), False),                       # 88.3, 85.5
    (dict(nx=155, ny=80, nu=61, nv=11, precision="fp32_store"), False),    # 83.4, 80.1
    (dict(nx=57, ny=20, nu=51, nv=28, precision="fp32_store"), False),     # 45.5, 43.2
    (dict(nx=70, ny=26, nu=11, nv=48, bc=0), False),                       # 46.1, 44.9
]


@pytest.mark.parametrize("form,by_node", MEASURED + list(zip(
    NODES.FORMS + MORE.FORMS, [True, True, True, True, False, True] + [True] * len(MORE.FORMS))),
    ids=str)
def test_which_solvers_split_their_update_chunks_by_node(program, form, by_node):
    assert ("update_kernel_nodes" in _kernels(program, **form)) == by_node


@pytest.mark.parametrize("form", FACES.FORMS, ids=str)
@pytest.mark.parametrize("mesh,faces,waves", list(zip(
    FACES.MESHES, [16, 16, 32, 64, 32, 64, 64], [8, 8, 8, 8, 8, 4, 8])), ids=str)
def test_which_interface_kernel_a_mesh_takes(program, mesh, faces, waves, form):
    names = _kernels(program, *mesh, 16, 18, **form)
    assert f"faces_kernel_chunksILi{faces}ELi{waves}E" in names
    assert names.count("faces_kernel") == 1
