"""The passes along y and x plane by plane, for every length that has them and the
next longer ones: the
product against the oracle, relative 1e-12 in FP64 and 2e-5 in c64, and against the
separate passes, 1e-14 sqrt(log2 P) and 1e-6 sqrt(log2 P) (a few roundings of each
transform, rms); one right-hand side (few planes, the widest work-groups), three and
seventeen; scatterers filling the padded grid (a sphere at its own length) and far
smaller than it; planar ones; and after a look at a stage, which runs the separate
passes on the same buffers."""

import functools
import math

import numpy as np
import pytest

from oracle import aim as oaim
from oracle.constants import wavenumber
from oracle.rwg import build_rwg
from workloads import plate_mesh, random_current, sphere_mesh

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

FREQ = 0.3e9
MESHES = {
    "sphere": lambda: sphere_mesh(0.4, FREQ, nf=3),
    "sphere1": lambda: sphere_mesh(1.0, FREQ, nf=6),
    "plate": lambda: plate_mesh(1.0, FREQ, jitter_seed=2),
}
LENGTHS = [21, 24, 27, 32, 36, 42, 48, 54, 63, 72, 81, 90, 96, 108, 112, 120, 126, 144, 162, 192,
           224, 252]


@functools.lru_cache(maxsize=None)
def _oracle(name):
    m = MESHES[name]()
    return m, oaim.build_operator(build_rwg(m.verts, m.tris), wavenumber(FREQ), 0.1 * m.lam, 2,
                                  0.3 * m.lam)


@functools.lru_cache(maxsize=None)
def _product(name, nrhs):
    _, op = _oracle(name)
    x = random_current(op.n, nrhs=nrhs, seed=nrhs)
    x = x.astype(np.complex64).astype(np.complex128)
    return x, oaim.matvec_fft(op, x)


@pytest.mark.parametrize("name,length", [("sphere", p) for p in LENGTHS] +
                         [("plate", p) for p in LENGTHS if p <= 96] + [("sphere1", 0)])
def test_product(name, length):
    from paper_1010_1456_amd import aim as A

    m, _ = _oracle(name)
    mesh = [(m.verts, m.tris, FREQ)]
    plan, sep = A.Plan(mesh, fft_min_pad=length), A.Plan(mesh, fft_min_pad=length, xy_groups=1)
    pad = plan.info()["pad"][0]
    assert pad[0] == pad[1] and pad[0] >= length
    few = math.sqrt(math.log2(pad[0]))
    for nrhs in (1, 3, 17):
        x, ref = _product(name, nrhs)
        xt = torch.from_numpy(x).cuda()
        for prec, inp, tol, close in ((A.AIM_FP64, xt, 1e-12, 1e-14 * few),
                                      (A.AIM_MIXED, xt.to(torch.complex64), 2e-5, 1e-6 * few)):
            y = plan.matvec(inp, prec)
            plan.product_stage(0, inp, 3, prec)
            assert torch.equal(plan.matvec(inp, prec), y)
            y = y.cpu().numpy().astype(np.complex128)
            z = sep.matvec(inp, prec).cpu().numpy().astype(np.complex128)
            for r in range(nrhs):
                nr = np.linalg.norm(ref[r])
                assert np.linalg.norm(y[r] - ref[r]) <= tol * nr, (nrhs, prec, r)
                assert np.linalg.norm(y[r] - z[r]) <= close * nr, (nrhs, prec, r)
