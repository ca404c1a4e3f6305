"""The passes along y and x plane by plane on planes filled with sources (P/2, for odd
P (P + 1)/2, nodes along both axes, so every row and column round of a work-group
runs and the last rows are reached), for every length that has them: coarse spheres
(P_z = P), plates between grid planes (third order, few planes) and plates in one;
few planes (the widest work-groups) and many. The propagated fields, as the product's
own passes leave them, against the separate passes: 1e-14 sqrt(log2 P) in FP64 and
1e-6 sqrt(log2 P) in c64 (a few roundings of each transform, rms; the product itself
is no measure here, since the interpolation onto these coarse meshes, wider than
their stencils, amplifies them). And which of the two a product takes."""

import math

import pytest

from workloads import plate_mesh, sphere_mesh

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

FREQ = 0.3e9
LENGTHS = [42, 48, 54, 63, 72, 81, 90, 96, 108, 112, 120, 126, 144, 162]


def _filling(shape, length, order):
    """A scatterer with ceil(length / 2) nodes along x and y (plates: the largest
    lambda/9 one with no more)."""
    from paper_1010_1456_amd import aim as A

    nodes = (length + 1) // 2
    if shape == "plate":
        squares = range(int(0.9 * nodes), 0, -1)
        tries = (plate_mesh(s / 9.0, FREQ) for s in squares)
    else:
        radii = (0.05 * (nodes - 3) + 0.004 * k for k in range(-30, 30))
        tries = (sphere_mesh(r, FREQ, nf=6) for r in radii)
    for m in tries:
        g = A.host_plan(m.verts, m.tris, FREQ, order=order, near_radius_lambda=0.0)["grid"]
        if g[0] == g[1] and (g[0] == nodes or (shape == "plate" and g[0] < nodes)):
            return m, g[0]
    raise AssertionError("no such scatterer")


@pytest.mark.parametrize("length", LENGTHS)
@pytest.mark.parametrize("shape,order", [("sphere", 2), ("plate", 3), ("plate", 2)])
def test_full_planes(shape, order, length):
    from paper_1010_1456_amd import aim as A

    m, nodes = _filling(shape, length, order)
    mesh = [(m.verts, m.tris, FREQ)]
    plan, sep = A.Plan(mesh, order=order), A.Plan(mesh, order=order, xy_groups=1)
    assert plan.info()["pad"][0][:2] == (length, length) and nodes >= (length + 1) // 2 - 1
    few = math.sqrt(math.log2(length))
    for nrhs in (1, 3, 16):
        if shape == "sphere" and nrhs == 16 and length > 96:
            continue
        x = torch.randn(nrhs, plan.n_total, dtype=torch.complex128, device="cuda",
                        generator=torch.Generator(device="cuda").manual_seed(length))
        for prec, inp, tol in ((A.AIM_FP64, x, 1e-14 * few),
                               (A.AIM_MIXED, x.to(torch.complex64), 1e-6 * few)):
            y = plan.product_stage(0, inp, 6, prec).to(torch.complex128).reshape(nrhs, -1)
            z = sep.product_stage(0, inp, 6, prec).to(torch.complex128).reshape(nrhs, -1)
            err = ((y - z).norm(dim=1) / z.norm(dim=1)).max().item()
            assert err <= tol, (nrhs, prec, err)
    plan.close()
    sep.close()


# (shape, order, length, FP64, right-hand sides): plane by plane
ROUTES = [("sphere", 2, 126, True, 1, True), ("sphere", 2, 126, True, 3, True),
          ("sphere", 2, 144, False, 3, True), ("sphere", 2, 144, True, 1, False),
          ("sphere", 2, 112, True, 1, True), ("sphere", 2, 112, True, 8, False),
          ("plate", 3, 126, True, 1, False), ("plate", 3, 112, True, 1, False),
          ("plate", 3, 112, True, 3, False), ("plate", 3, 108, True, 1, False),
          ("plate", 3, 108, True, 3, True), ("plate", 3, 126, False, 1, True),
          ("plate", 3, 162, False, 1, False), ("plate", 3, 162, False, 3, True),
          ("plate", 2, 90, False, 1, True), ("plate", 2, 90, True, 1, False),
          ("plate", 2, 81, True, 1, True), ("plate", 2, 96, False, 16, False)]


@pytest.mark.parametrize("shape,order,length,fp64,nrhs,planes", ROUTES)
def test_route(shape, order, length, fp64, nrhs, planes):
    from torch.profiler import ProfilerActivity, profile

    from paper_1010_1456_amd import aim as A

    m, _ = _filling(shape, length, order)
    plan = A.Plan([(m.verts, m.tris, FREQ)], order=order, tune_rhs=nrhs)
    x = torch.ones(nrhs, plan.n_total, dtype=torch.complex128 if fp64 else torch.complex64,
                   device="cuda")
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        plan.matvec(x, A.AIM_FP64 if fp64 else A.AIM_MIXED)
        torch.cuda.synchronize()
    names = [e.name for e in prof.events()]
    assert any("k_fft_plane" in s for s in names) == planes, names
    assert any("k_fft_mid" in s for s in names) != planes, names
    plan.close()
