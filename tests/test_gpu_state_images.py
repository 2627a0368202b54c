"""Host images of the distribution: states of one piece, of many pieces (several host threads), of
cells that need several pieces each, and both storage types go to the solver and back unchanged,
and a solver set to another's state steps on to the same bits."""
import numpy as np
import pytest

from paper_1810_08137_amd import ugks
from paper_1810_08137_amd import workloads as WL

pytestmark = pytest.mark.gpu

CASES = [
    dict(nx=1, ny=1, nu=2, nv=3),                       # a few values
    dict(nx=65, ny=3, nu=9, nv=7, dof=1),               # ragged tiles, two distributions
    dict(nx=63, ny=2, nu=8, nv=8, bc=0),
    dict(nx=3, ny=2, nu=520, nv=507),                   # a cell is more than one piece
    dict(nx=43, ny=31, nu=64, nv=61),                   # 20 pieces, the last one short
    dict(nx=43, ny=31, nu=64, nv=61, precision="fp32_store"),
]


@pytest.mark.parametrize("form", CASES, ids=lambda f: "-".join(str(v) for v in f.values()))
def test_state_goes_out_and_back(form):
    case = dict(WL.CHANNEL_DEFAULTS, lx=2.0, ly=1.0, umax=5.0, vmax=5.0, kn=0.1, seed=3)
    case.update(form)
    precision = case.pop("precision", "fp64")
    kn, kw = WL.solver_kwargs(case, precision)
    a, b = ugks.Solver(kn, **kw), ugks.Solver(kn, **kw)
    f0, W0 = a.state()
    rng = np.random.default_rng(1)
    f = f0 * (1.0 + 0.01 * rng.uniform(-1.0, 1.0, f0.shape))
    a.set_state(f, W0)
    fa, Wa = a.state()
    want = f.astype(np.float32).astype(np.float64) if precision == "fp32_store" else f
    assert np.array_equal(fa, want) and np.array_equal(Wa, W0)
    if case["nu"] > 2:
        a.step(2)
        b.set_state(f, W0)
        b.step(2)
        for x, y in zip(a.state(), b.state()):
            assert np.array_equal(x, y)
    a.close()
    b.close()


@pytest.mark.parametrize("mesh", [(1, 1), (7, 5), (300, 219)], ids=str)
def test_moments_are_those_of_the_state(mesh):
    """(300 x 219 cells: more than one piece.)  The primitive variables of W, operation by
    operation, so the values are the same bits."""
    case = dict(WL.CHANNEL_DEFAULTS, nx=mesh[0], ny=mesh[1], lx=2.0, ly=1.0, nu=8, nv=8, umax=4.0,
                vmax=4.0, kn=0.1, seed=4, dof=1)
    kn, kw = WL.solver_kwargs(case, "fp64")
    s = ugks.Solver(kn, **kw)
    s.step(2)
    _, W = ugks.ugks_get_state(s.h, want_f=False)
    m = s.moments()
    rho, U, V = W[..., 0], W[..., 1] / W[..., 0], W[..., 2] / W[..., 0]
    T = (W[..., 3] - 0.5 * rho * (U * U + V * V)) / (0.75 * rho)
    assert np.array_equal(m, np.stack([rho, U, V, T], -1))
    # an invalid cell anywhere is reported, after the values are written
    W[-1, -1, 3] = -1.0
    s.set_state(W=W)
    with pytest.raises(ugks.UgksError) as e:
        s.moments()
    assert e.value.code == ugks.UGKS_E_STATE
    s.close()
