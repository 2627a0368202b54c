"""The workspace and the transient buffers of a step hold what the layout documents and no more: narrow
meshes, where a row's two ghost cells weigh most, keep the size (and with it ugks_step_static, whose
scratch is fixed) that they have with each ghost cell's 17 sums kept apart.  CPU only; that
ugks_step_static takes such a shape is the case `static_scratch` of tests/host."""
import pytest

from paper_1810_08137_amd import ugks
from paper_1810_08137_amd import workloads as WL

SHAPES = [
    dict(nx=1, ny=3000, nu=2, nv=2),
    dict(nx=4, ny=10000, nu=2, nv=2),
    dict(nx=4, ny=500, nu=8, nv=8, bc=0),
    dict(nx=2, ny=700, nu=9, nv=6, prandtl=2.0 / 3.0),
    dict(nx=3, ny=400, nu=12, nv=6, dof=2, precision="fp32_store"),
    dict(nx=40, ny=20, nu=29, nv=29),
]


def transient_bytes(nx, ny, G, NC, shak):
    cells, xf, yf = nx * ny, ny * (nx + 1), (ny + 1) * nx
    sums = NC * G * (cells * (76 if shak else 64) + 2 * ny * 17)
    return 8 * (sums + NC * 32 * (xf + yf))


@pytest.mark.parametrize("form", SHAPES, ids=lambda f: "-".join(str(v) for v in f.values()))
def test_workspace_holds_no_more_than_its_buffers(form):
    c = dict(WL.CHANNEL_DEFAULTS, lx=1.0, ly=1.0, umax=5.0, vmax=5.0)
    c.update(form)
    mesh, vgrid, _, opts = ugks.make_structs(**c)
    nx, ny, K, M = c["nx"], c["ny"], c["nu"], c["nv"]
    NC = 2 if c.get("dof") else 1
    shak = 0 < c.get("prandtl", 1.0) < 1
    ss = 4 if c.get("precision") == "fp32_store" else 8
    G = max(1, min(3 * 256 // (-(-nx // 60) * ny * NC), K // 2, 16))
    plane = -(-((nx + 4) * (ny + 4)) // 64) * 64
    documented = (2 * NC * K * M * plane * ss + 2 * 4 * 8 * nx * ny + 2 * 4 * 8 * ny
                  + transient_bytes(nx, ny, G, NC, shak) + 8 * (2 * K + 7 * M + ny))
    small = 16 << 10   # flags, two launch plans, the alignment of each buffer
    need = ugks.ugks_required_bytes(mesh, vgrid, opts)
    assert documented <= need + 8 * NC * G * 2 * ny      # no heat sums without Shakhov
    assert need <= documented + small
