"""Update-kernel chunks by node in every form of that kernel: the same bits as in a batch (whole
lines), and the oracle's values.  tests/test_host_runtime.py checks that all of these solvers take
it."""
import numpy as np
import pytest

from paper_1810_08137_amd import ugks
from tests import parity as PR
from tests.test_gpu_update_nodes import _case, _solver

pytestmark = pytest.mark.gpu

FORMS = [
    dict(nx=40, ny=20, nu=29, nv=9),                           # five nodes in a line
    dict(nx=26, ny=39, nu=47, nv=21),                          # odd rows, two chunks a workgroup
    dict(nx=70, ny=16, nu=34, nv=22, bc=0),
    dict(nx=66, ny=7, nu=49, nv=21, dof=1),
    dict(nx=33, ny=5, nu=40, nv=11, dof=1),                    # one chunk a workgroup
    dict(nx=95, ny=37, nu=41, nv=10, bc=0, precision="fp32_store"),
]
IDS = ["short lines", "odd rows", "periodic", "dof", "dof, one chunk", "periodic fp32"]


@pytest.mark.parametrize("form", FORMS, ids=IDS)
def test_chunks_by_node_change_no_result(form):
    case, precision = _case(form)
    alone, member, other = (_solver(case, precision) for _ in range(3))
    batch = ugks.Batch(2)
    alone.step(4)
    batch.step([member, other], 4)
    for a, b in zip(alone.state(), member.state()):
        assert np.array_equal(a, b)
    for s in (alone, member, other):
        s.close()
    batch.close()


@pytest.mark.parametrize("form", FORMS, ids=IDS)
def test_chunks_by_node_match_the_oracle(form):
    case, precision = _case(form)
    tol = PR.FP64_TOL if precision == "fp64" else PR.FP32_STORE_TOL
    PR.run_and_compare(case, 3, precision=precision, tol=tol, label=f"by node {form}")
