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
from oracle.constants import ETA0, wavenumber
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


def _sigma_extended(rwg, verts, k, x, th, ph):
    """sigma_tt by the 7-point rule of every triangle in extended precision."""
    L = np.longdouble
    s15 = np.sqrt(L(15))
    weights = [L(9) / 40] + [(155 - s15) / 1200] * 3 + [(155 + s15) / 1200] * 3
    bary = [[L(1) / 3] * 3] + [[1 - 2 * a if c == p else a for c in range(3)]
                               for a in ((6 - s15) / 21, (6 + s15) / 21) for p in range(3)]
    V = verts.astype(L)
    T = V[rwg.tris]
    area = np.sqrt((np.cross(T[:, 1] - T[:, 0], T[:, 2] - T[:, 0]) ** 2).sum(1)) / 2
    pts = np.stack([sum(b[c] * T[:, c] for c in range(3)) for b in bary], 1)
    J = np.zeros(pts.shape, dtype=np.clongdouble)
    length = np.sqrt(((V[rwg.edge[:, 1]] - V[rwg.edge[:, 0]]) ** 2).sum(1))
    for s, t, v in ((1, rwg.tplus, rwg.vplus), (-1, rwg.tminus, rwg.vminus)):
        f = (s * length / (2 * area[t])) * x.astype(np.clongdouble)
        np.add.at(J, t, f[:, None, None] * (pts[t] - V[v][:, None]))
    wt = np.array(weights) * area[:, None]
    scale = (L(k) * L(ETA0)) ** 2 / (4 * L("3.14159265358979323846264338327950288"))
    out = np.empty((len(th), len(ph)), dtype=L)
    for i, a in enumerate(th.astype(L)):
        for j, b in enumerate(ph.astype(L)):
            rh = np.array([np.sin(a) * np.cos(b), np.sin(a) * np.sin(b), np.cos(a)])
            tt = np.array([np.cos(a) * np.cos(b), np.cos(a) * np.sin(b), -np.sin(a)])
            p = L(k) * (pts @ rh)
            out[i, j] = scale * abs(((J @ tt) * wt * (np.cos(p) + 1j * np.sin(p))).sum()) ** 2
    return out


@pytest.mark.parametrize("current", ["random", "wave"])
def test_rounding_of_the_phases(current):
    """An 8-lambda plate against extended precision, rms relative to the rms sigma: each
    phase is rounded a handful of times by up to half an ulp of 4 wavelengths, 2.8e-15
    radians, alike along a grid line (72 lines): 2 x 2.8e-15 x sqrt(3 / 72) = 1.2e-15.
    (A rounded k / 6 pi, the sum of the corners rounded before it and the edge vectors
    taken from the centroid gave 2.2e-15 and 5.5e-15.)"""
    from paper_1010_1456_amd import aim as A

    m = plate_mesh(8.0, FREQ)
    rwg = build_rwg(m.verts, m.tris)
    k = wavenumber(FREQ)
    x = (random_current(rwg.n, nrhs=1, seed=3)[0] if current == "random"
         else np.exp(1j * k * rwg.centre[:, 0]))
    th, ph = np.linspace(0.1, 3.0, 7), np.linspace(0.0, 6.0, 6)
    ref = _sigma_extended(rwg, m.verts, k, x, th, ph)
    plan = A.Plan([(m.verts, m.tris, FREQ)], mixed=False)
    got = plan.rcs(torch.from_numpy(x).cuda()[None], th, ph)[0, 0]
    plan.close()
    err = np.sqrt(((got.astype(np.longdouble) - ref) ** 2).sum() / (ref**2).sum())
    assert err <= 1.2e-15


@pytest.mark.parametrize("ntheta,nphi,nrhs,wide", [
    (1, 1, 17, 1), (2, 128, 16, 2), (4, 128, 16, 4), (8, 128, 5, 4), (8, 128, 9, 8),
    (8, 128, 17, 16), (91, 180, 17, 16)])
def test_work_split(ntheta, nphi, nrhs, wide):
    """Few directions are summed in shorter chunks and, if that gives too few
    work-groups, with fewer right-hand sides in each: every width, also where the
    scratch of the interface without allocation limits the chunks."""
    from torch.profiler import ProfilerActivity, profile

    from paper_1010_1456_amd import aim as A

    m = plate_mesh(2.0, FREQ, jitter_seed=5)  # 648 triangles
    rwg = build_rwg(m.verts, m.tris)
    plan = A.Plan([(m.verts, m.tris, FREQ)], mixed=False)
    x = random_current(rwg.n, nrhs=nrhs, seed=nrhs)
    th = np.linspace(0.1, math.pi - 0.1, ntheta)
    ph = np.linspace(0.0, 2.0 * math.pi, nphi, endpoint=False) + 0.1
    xt, dth, dph = (torch.from_numpy(v).cuda() for v in (x, th, ph))
    got = [plan.rcs(xt, th, ph)[0]]
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        got.append(plan.rcs_noalloc(xt, dth, dph)[0].cpu().numpy())
    assert any(f"k_rcs_part<{wide}>" in e.name for e in prof.events())
    rows = [0, ntheta // 2, ntheta - 1]
    for r in (0, nrhs // 2, nrhs - 1):
        ref = off.sigma_tt(rwg, wavenumber(FREQ), x[r], th[rows], ph)
        for g in got:
            assert np.abs(g[r][rows] - ref).max() <= 1e-12 * np.abs(g[r]).max(), r
    plan.close()
