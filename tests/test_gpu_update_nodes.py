"""Update-kernel chunks that split a quadrant's nodes instead of its u lines: chosen for a solver
alone where the lines do not divide evenly over its chunks, never in a batch.  The split changes
no result: alone and in a batch the states are the same bit for bit, and alone they match the
oracle within the FP64 (FP32-storage) bar."""
import numpy as np
import pytest

from paper_1810_08137_amd import ugks
from paper_1810_08137_amd import workloads as WL
from tests import parity as PR

pytestmark = pytest.mark.gpu

# velocity grids with odd halves, fewer nodes in a line than a group of three, chunks that start
# and end inside lines, v halves in chunks of their own (small meshes), odd rows
FORMS = [
    dict(nx=40, ny=20, nu=29, nv=29),
    dict(nx=40, ny=20, nu=29, nv=8),
    dict(nx=80, ny=40, nu=25, nv=13, precision="fp32_store"),
    dict(nx=61, ny=7, nu=33, nv=20, dof=1),
    dict(nx=120, ny=31, nu=49, nv=11, bc=0),
    dict(nx=25, ny=9, nu=43, nv=31, precision="fp32_store", dof=2),
]


def _case(form):
    c = dict(WL.CHANNEL_DEFAULTS, lx=2.0, ly=1.0, umax=5.0, vmax=5.0, kn=0.1, seed=11)
    c.update(form)
    return c, c.pop("precision", "fp64")


def _solver(case, precision):
    kn, kw = WL.solver_kwargs(case, precision)
    return ugks.Solver(kn, **kw)


@pytest.mark.parametrize("form", FORMS, ids=lambda f: "-".join(str(v) for v in f.values()))
def test_chunks_by_node_change_no_result(form):
    case, precision = _case(form)
    alone, member, other = (_solver(case, precision) for _ in range(3))
    batch = ugks.Batch(2)
    alone.step(4)
    batch.step([member, other], 4)
    fa, Wa = alone.state()
    fb, Wb = member.state()
    assert np.array_equal(fa, fb)
    assert np.array_equal(Wa, Wb)
    for s in (alone, member, other):
        s.close()
    batch.close()


@pytest.mark.parametrize("form", FORMS, ids=lambda f: "-".join(str(v) for v in f.values()))
def test_chunks_by_node_match_the_oracle(form):
    case, precision = _case(form)
    tol = PR.FP64_TOL if precision == "fp64" else PR.FP32_STORE_TOL
    PR.run_and_compare(case, 3, precision=precision, tol=tol, label=f"by node {form}")


def test_a_batch_in_any_order_steps_as_alone():
    """A plan takes its instances in the order of their velocity counts: whatever order the
    caller's list has, every member steps to the bits it has alone."""
    shapes = [(50, 12, 24), (61, 7, 48), (9, 3, 32), (100, 25, 24), (1, 1, 48), (130, 5, 33)]
    alone, members = [], []
    for n, (nx, ny, nv) in enumerate(shapes):
        case = dict(WL.CHANNEL_DEFAULTS, lx=2.0, ly=1.0, umax=5.0, vmax=5.0, kn=0.1, seed=n,
                    nx=nx, ny=ny, nu=nv, nv=nv, bc=n % 2)
        alone.append(_solver(case, "fp64"))
        members.append(_solver(case, "fp64"))
    batch = ugks.Batch(len(shapes))
    for order in ([0, 1, 2, 3, 4, 5], [5, 3, 1, 4, 2, 0], [2, 5]):
        batch.step([members[k] for k in order], 2)
        for k in order:
            alone[k].step(2)
    for a, b in zip(alone, members):
        for x, y in zip(a.state(), b.state()):
            assert np.array_equal(x, y)
        a.close()
        b.close()
    batch.close()
