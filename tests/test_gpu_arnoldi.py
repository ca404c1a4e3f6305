"""The Arnoldi step where its kernels change: the iterate after k steps of one
cycle against the oracle's GMRES at the same k, FP64, for k around the basis
tiles (16, 32, 64, 112, 208 vectors) and the 8-step segments, rows that are no
multiple of a tile, one and three right-hand sides, restarted cycles, captured
and launched directly. The iterates agree to k kappa eps: kappa is about 1e4 here,
so 1e-9 relative."""

import functools

import numpy as np
import pytest

from oracle import aim as oaim
from oracle import excitation as oexc
from oracle import gmres as ogmres
from oracle.constants import wavenumber
from oracle.rwg import build_rwg
from workloads import plate_mesh

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

FREQ = 0.3e9
WAVES = [(0.4, 0.3, 0), (0.9, 2.0, 1), (0.0, 0.0, 0)]


@functools.lru_cache(maxsize=None)
def _problem(side):
    from paper_1010_1456_amd import aim as A

    m = plate_mesh(side, FREQ, jitter_seed=7)
    rwg = build_rwg(m.verts, m.tris)
    k = wavenumber(FREQ)
    op = oaim.build_operator(rwg, k, 0.1 * m.lam, 2, 0.3 * m.lam)
    return rwg, k, op, A.Plan([(m.verts, m.tris, FREQ)], mixed=False)


@functools.lru_cache(maxsize=None)
def _reference(side, wave, steps, restart):
    rwg, k, op, _ = _problem(side)
    b = oexc.planewave_rhs(rwg, k, *WAVES[wave])
    x, st = ogmres.gmres(lambda v: oaim.matvec_fft(op, v), b, op.zmom_diag, 1e-15,
                         restart=restart, max_iter=steps)
    assert st["iters"] == steps
    return x


@pytest.mark.parametrize("graphs", [True, False])
@pytest.mark.parametrize("side,nrhs,steps,restart", [
    (1.0, 1, 1, 5), (1.0, 3, 8, 8), (1.0, 1, 13, 40), (1.0, 2, 16, 16), (1.0, 1, 17, 17),
    (2.0, 1, 33, 40), (2.0, 3, 34, 34), (2.0, 1, 65, 80), (2.0, 1, 113, 200), (2.0, 3, 120, 130),
    (1.0, 2, 33, 33), (1.0, 1, 66, 90), (1.0, 1, 98, 100), (2.0, 1, 30, 9), (1.0, 3, 29, 12),
    (4.5, 1, 20, 25), (4.5, 2, 66, 70), (2.0, 2, 129, 129), (2.0, 1, 196, 200),
])
def test_iterate_after_k_steps(side, nrhs, steps, restart, graphs):
    from paper_1010_1456_amd import aim as A

    _, _, _, plan = _problem(side)
    for _ in range(2):  # the second solve replays the first one's graphs
        x, st = plan.solve(WAVES[:nrhs], A.AIM_FP64, tol=1e-15, restart=restart, max_iter=steps,
                           raise_on_noconv=False, graphs=graphs)
        assert all(s["iterations"] == steps for s in st)
        for r in range(nrhs):
            ref = _reference(side, r, steps, restart)
            got = x[r].cpu().numpy()
            assert np.linalg.norm(got - ref) <= 1e-9 * np.linalg.norm(ref), r
