"""The far-field kernel against the oracle where its shapes change: right-hand
sides around its 1, 2, 4, 8 and 16-wide variants, directions around its
128-direction groups, triangles on both sides of the size up to which their
phase is summed as a series (about lambda/6.5 here) and far above it, and a
scatterer far from the origin. Both interfaces, FP64, 1e-12 of the largest
sigma (1e-11 for the displaced one, whose phases of about 6e3 radians carry
1e-12 each)."""

import math

import numpy as np
import pytest

from oracle import farfield as off
from oracle.constants import wavenumber
from oracle.rwg import build_rwg
from workloads import plate_mesh, random_current, sphere_mesh

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

FREQ = 0.3e9


def _check(verts, tris, freq, nrhs, ntheta, nphi, tol):
    from paper_1010_1456_amd import aim as A

    rwg = build_rwg(verts, tris)
    k = wavenumber(freq)
    plan = A.Plan([(verts, tris, freq)], mixed=False)
    try:
        x = random_current(rwg.n, nrhs=nrhs, seed=nrhs)
        th = np.linspace(0.0, math.pi, ntheta)
        ph = np.linspace(0.0, 2.0 * math.pi, nphi, endpoint=False) + 0.1
        ref = np.stack([off.sigma_tt(rwg, k, x[r], th, ph) for r in range(nrhs)])
        xt = torch.from_numpy(x).cuda()
        got = plan.rcs(xt, th, ph)[0]
        dev = plan.rcs_noalloc(xt, torch.from_numpy(th).cuda(), torch.from_numpy(ph).cuda())
        for r in range(nrhs):
            for g in (got[r], dev[0, r].cpu().numpy()):
                err = np.abs(g - ref[r]).max() / np.abs(ref[r]).max()
                assert err <= tol, (r, err)
    finally:
        plan.close()


@pytest.mark.parametrize("nrhs", [1, 2, 3, 5, 9, 16, 17, 35])
def test_right_hand_sides(nrhs):
    m = sphere_mesh(0.5, FREQ, nf=4)
    _check(m.verts, m.tris, FREQ, nrhs, 7, 5, 1e-12)


@pytest.mark.parametrize("ntheta,nphi", [(1, 1), (1, 127), (16, 8), (43, 3), (3, 86)])
def test_directions(ntheta, nphi):
    m = plate_mesh(2.0, FREQ, jitter_seed=5)  # several triangle batches and chunks
    _check(m.verts, m.tris, FREQ, 2, ntheta, nphi, 1e-12)


@pytest.mark.parametrize("squares_per_lambda", [7, 6, 2, 1])
def test_triangle_sizes(squares_per_lambda):
    m = plate_mesh(2.0, FREQ, squares_per_lambda=squares_per_lambda)
    _check(m.verts, m.tris, FREQ, 3, 19, 12, 1e-12)


def test_displaced_scatterer():
    m = sphere_mesh(0.5, FREQ, nf=5)
    _check(m.verts + np.array([700.0, -600.0, 300.0]), m.tris, FREQ, 1, 9, 7, 1e-11)
