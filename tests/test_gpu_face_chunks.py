"""The interface kernel of solvers whose moment kernel leaves several parts of every sum: its forms
(16, 32 or 64 faces a workgroup, eight or four wavefronts, by the number of faces) on meshes at
both sides of the limits, each with several velocity chunks.  Alone they match the oracle within
the FP64 bar, and a batch (which takes another form, by all its members' faces) steps them to
the same bits."""
import numpy as np
import pytest

from paper_1810_08137_amd import ugks
from paper_1810_08137_amd import workloads as WL
from tests import parity as PR

pytestmark = pytest.mark.gpu

# (nx, ny): faces ny (nx + 1) + (ny + 1) nx
MESHES = [
    (7, 3),      # less than one workgroup of either family
    (45, 43),    # 3956: 16 faces, the last such size
    (60, 33),    # 4053: 32 faces, the first
    (61, 65),    # 8056: 64 faces
    (57, 69),    # 7992: 32 faces, the last such size
    (120, 66),   # 16026: 64 faces, four wavefronts
    (117, 67),   # 15862: 64 faces, eight wavefronts
]
FORMS = [dict(), dict(prandtl=2.0 / 3.0), dict(dof=1), dict(bc=0)]


def _case(mesh, form):
    c = dict(WL.CHANNEL_DEFAULTS, lx=2.0, ly=1.0, umax=5.0, vmax=5.0, kn=0.1, seed=13,
             nx=mesh[0], ny=mesh[1], nu=16, nv=18)
    c.update(form)
    return c


def _solver(case):
    kn, kw = WL.solver_kwargs(case)
    return ugks.Solver(kn, **kw)


@pytest.mark.parametrize("form", FORMS, ids=["bgk", "shakhov", "dof", "periodic"])
@pytest.mark.parametrize("mesh", MESHES, ids=lambda m: f"{m[0]}x{m[1]}")
def test_sums_in_parts(mesh, form):
    case = _case(mesh, form)
    PR.run_and_compare(case, 2, label=f"sums in parts {mesh} {form}")
    alone, member, other = _solver(case), _solver(case), _solver(_case((130, 70), form))
    assert alone.info.moment_chunks > 1
    batch = ugks.Batch(2)
    alone.step(3)
    batch.step([other, member], 3)
    fa, Wa = alone.state()
    fb, Wb = member.state()
    assert np.array_equal(fa, fb)
    assert np.array_equal(Wa, Wb)
    for s in (alone, member, other):
        s.close()
    batch.close()
