"""The near-zone fill against the oracle where its shapes change: rows with more
entries than a batch and more triangles than one batch holds (halved batches),
more stencil nodes than one pass holds, a node box too large for the per-row
kernel (the double sum per entry), the in-plane stencil of a plate, odd orders,
EFIE and CFIE. Matrix and diagonal to 1e-12 of their largest entry."""

import numpy as np
import pytest

from oracle import aim as oaim
from oracle.constants import wavenumber
from oracle.rwg import build_rwg
from workloads import plate_mesh, sphere_mesh

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

FREQ = 0.3e9

CASES = {
    # ~120 and all 270 entries per row, 180 triangles, up to 1 331 nodes
    "sphere_wide": (lambda: sphere_mesh(0.5, FREQ, nf=3), 2, 0.55, 0.6),
    "sphere_all": (lambda: sphere_mesh(0.5, FREQ, nf=3), 2, 1.1, 0.6),
    "sphere_all_efie": (lambda: sphere_mesh(0.5, FREQ, nf=3, jitter_seed=3), 3, 1.1, None),
    # reach 13 on a 17-node grid: 29^3 cells
    "sphere_box": (lambda: sphere_mesh(0.8, FREQ, nf=3), 2, 1.3, 0.6),
    "sphere_box_efie": (lambda: sphere_mesh(0.8, FREQ, nf=3), 2, 1.3, None),
    "plate_wide": (lambda: plate_mesh(1.0, FREQ, jitter_seed=4), 2, 0.8, None),
    "plate_odd": (lambda: plate_mesh(1.0, FREQ), 3, 0.4, None),
    # no neighbour but the basis itself
    "plate_self": (lambda: plate_mesh(1.0, FREQ), 2, 0.0, None),
}


@pytest.mark.parametrize("name", list(CASES))
def test_near_matrix(name):
    from paper_1010_1456_amd import aim as A

    make, order, radius, alpha = CASES[name]
    m = make()
    rwg = build_rwg(m.verts, m.tris)
    kw = {} if alpha is None else {"cfie_alpha": alpha}
    op = oaim.build_operator(rwg, wavenumber(FREQ), 0.1 * m.lam, order, radius * m.lam, **kw)
    plan = A.Plan([(m.verts, m.tris, FREQ)], order=order, near_radius_lambda=radius, mixed=False, **kw)
    try:
        near = plan.export(0, A.AIM_DATA_NEAR64)
        ref = op.near.data
        assert near.shape == ref.shape
        assert np.abs(near - ref).max() <= 1e-12 * np.abs(ref).max()
        zd = plan.export(0, A.AIM_DATA_ZDIAG64)
        assert np.abs(zd - op.zmom_diag).max() <= 1e-12 * np.abs(op.zmom_diag).max()
    finally:
        plan.close()


# the per-row kernel with more than 64 KB of LDS, up to its bounds, and the first
# reach beyond them: boxes of 23^3, 25^3 and 27^3 nodes; in one grid plane of 89^2,
# 113^2 and 115^2
WIDE = {
    "box_reach_10": (lambda: sphere_mesh(0.8, FREQ, nf=3), 0.9, 0.6),
    "box_reach_11": (lambda: sphere_mesh(0.8, FREQ, nf=3), 1.0, 0.6),
    "box_reach_11_efie": (lambda: sphere_mesh(0.8, FREQ, nf=3), 1.0, None),
    "box_reach_12": (lambda: sphere_mesh(0.8, FREQ, nf=3), 1.1, 0.6),
    "plane_reach_43": (lambda: plate_mesh(6.2, FREQ, squares_per_lambda=1), 4.25, None),
    "plane_reach_55": (lambda: plate_mesh(6.2, FREQ, squares_per_lambda=1), 5.45, None),
    "plane_reach_56": (lambda: plate_mesh(6.2, FREQ, squares_per_lambda=1), 5.55, None),
}


@pytest.mark.parametrize("name", list(WIDE))
def test_wide_near_zone(name):
    from paper_1010_1456_amd import aim as A

    make, radius, alpha = WIDE[name]
    m = make()
    kw = {} if alpha is None else {"cfie_alpha": alpha}
    op = oaim.build_operator(build_rwg(m.verts, m.tris), wavenumber(FREQ), 0.1 * m.lam, 2,
                             radius * m.lam, **kw)
    plan = A.Plan([(m.verts, m.tris, FREQ)], near_radius_lambda=radius, mixed=False, **kw)
    try:
        reach = int(name.split("_")[2])
        info = plan.info()
        assert min(info["grid"][0][:2]) - 3 >= reach
        assert (info["planar_z"][0] >= 0) == name.startswith("plane")
        near = plan.export(0, A.AIM_DATA_NEAR64)
        ref = op.near.data
        assert near.shape == ref.shape
        assert np.abs(near - ref).max() <= 1e-12 * np.abs(ref).max()
    finally:
        plan.close()
