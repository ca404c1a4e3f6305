"""Set-up of more unknowns than one launch of the near-zone kernels has rows for: a
plate of 2 366 x 2 366 squares (16 789 136 unknowns, so n work-groups of 256 threads
are more than the 2^32 - 1 threads of a launch), first-order stencils, no near pair
but the basis itself. Rows around every boundary between launches, and the first
and last ones: Z^MOM's diagonal against the oracle's on a plate of the same squares
(the three edge directions), and the stored Z^MOM - Z^grid against it and the
exported weights, to 1e-9 (the coordinates are rounded at 2 366 times a square)."""

import numpy as np
import pytest

from oracle import aim as oaim
from oracle.constants import ETA0, wavenumber
from oracle.rwg import build_rwg
from workloads import plate_mesh

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

FREQ = 0.3e9
SQUARES = 2366
PER_LAMBDA = 40


def _directions(n):
    """0 (along x), 1 (along y) or 2 (diagonal) of each interior edge of an n x n
    plate, in the library's order: by the lower vertex, then the other one."""
    j, i = np.meshgrid(np.arange(n + 1), np.arange(n + 1), indexing="ij")
    has = np.stack([(i < n) & (0 < j) & (j < n), (j < n) & (0 < i) & (i < n), (i < n) & (j < n)], -1)
    return np.broadcast_to(np.arange(3, dtype=np.int8), has.shape)[has]


def test_rows_beyond_one_launch():
    from paper_1010_1456_amd import aim as A

    small = plate_mesh(8 / PER_LAMBDA, FREQ, squares_per_lambda=PER_LAMBDA)
    k, h = wavenumber(FREQ), 0.1 * small.lam
    op = oaim.build_operator(build_rwg(small.verts, small.tris), k, h, 1, 0.0)
    diag = np.array([op.zmom_diag[_directions(8) == d].mean() for d in range(3)])

    m = plate_mesh(SQUARES / PER_LAMBDA, FREQ, squares_per_lambda=PER_LAMBDA)
    plan = A.Plan([(m.verts, m.tris, FREQ)], order=1, near_radius_lambda=0.0, mixed=False)
    n, info = plan.n_total, plan.info()
    assert n == 3 * SQUARES**2 - 2 * SQUARES and 256 * n > 2**32
    assert info["nnz"][0] == n  # one entry per row: entry m is row m's
    zd = plan.export(0, A.AIM_DATA_ZDIAG64)
    near = plan.export(0, A.AIM_DATA_NEAR64)
    lam = plan.export(0, A.AIM_DATA_LAMBDA64)
    plan.close()
    ref = diag[_directions(SQUARES)]
    assert np.abs(zd - ref).max() <= 1e-9 * np.abs(diag).max()

    cuts = [0, n] + list(range(1 << 20, n, 1 << 20))
    rows = np.unique(np.concatenate([np.arange(max(c - 200, 0), min(c + 200, n)) for c in cuts]))
    u = np.stack(np.meshgrid(*[np.arange(2)] * 3, indexing="ij"), -1).reshape(-1, 3)
    r = h * np.linalg.norm(u[:, None] - u[None], axis=-1)
    g = np.where(r > 0, np.exp(-1j * k * r) / (4 * np.pi * np.where(r > 0, r, 1.0)), 0.0)
    q = np.einsum("mqu,uv,mqv->mq", lam[rows], g, lam[rows])
    zgrid = 1j * k * ETA0 * (q[:, :3].sum(1) - q[:, 3] / k**2)
    assert np.abs(near[rows] - (ref[rows] - zgrid)).max() <= 1e-9 * np.abs(diag).max()
