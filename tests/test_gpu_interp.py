"""The interpolation and near-zone kernel where its shapes change: right-hand
sides in groups of 4 and the 1 to 3 left over, a lane each from 6 on (8 or 16 lanes,
one or more groups of them), rows longer than one pass of 96
entries, stencils of up to 216 nodes, row counts that are no multiple of a
work-group's 16, in both arithmetics, against the oracle: relative 1e-12 in FP64,
2e-5 in c64, and the c128-vector form of the c64 product equal to it bit for bit
on c64-valued input."""

import functools

import numpy as np
import pytest

from oracle import aim as oaim
from oracle.constants import ETA0, wavenumber
from oracle.rwg import build_rwg
from workloads import plate_mesh, random_current, sphere_mesh

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

FREQ = 0.3e9

CASES = {
    "plate": (lambda: plate_mesh(1.0, FREQ), 2, 0.3, None),
    "sphere_long_rows": (lambda: sphere_mesh(0.5, FREQ, nf=4), 2, 0.5, 0.6),
    "plate_long_rows": (lambda: plate_mesh(1.0, FREQ, jitter_seed=2), 1, 0.8, None),
    "sphere_m3": (lambda: sphere_mesh(0.4, FREQ, nf=3), 3, 0.3, 0.6),
    "sphere_m5": (lambda: sphere_mesh(0.4, FREQ, nf=3), 5, 0.3, None),
}


@functools.lru_cache(maxsize=None)
def _problem(name):
    from paper_1010_1456_amd import aim as A

    make, order, radius, alpha = CASES[name]
    m = make()
    kw = {} if alpha is None else {"cfie_alpha": alpha}
    op = oaim.build_operator(build_rwg(m.verts, m.tris), wavenumber(FREQ), 0.1 * m.lam, order,
                             radius * m.lam, **kw)
    return op, A.Plan([(m.verts, m.tris, FREQ)], order=order, near_radius_lambda=radius, **kw)


@pytest.mark.parametrize("nrhs", [1, 2, 3, 4, 5, 6, 8, 9, 16, 17])
@pytest.mark.parametrize("name", list(CASES))
def test_product(name, nrhs):
    from paper_1010_1456_amd import aim as A

    op, plan = _problem(name)
    x = random_current(plan.n_total, nrhs=nrhs, seed=nrhs).astype(np.complex64).astype(np.complex128)
    ref = oaim.matvec_fft(op, x)
    xt = torch.from_numpy(x).cuda()
    y64 = plan.matvec(xt, A.AIM_FP64).cpu().numpy()
    y32 = plan.matvec(xt.to(torch.complex64), A.AIM_MIXED)
    yio = plan.matvec(xt, A.AIM_MIXED_IO64)
    for r in range(nrhs):
        nr = np.linalg.norm(ref[r])
        assert np.linalg.norm(y64[r] - ref[r]) <= 1e-12 * nr, r
        assert np.linalg.norm(y32[r].cpu().numpy() - ref[r]) <= 2e-5 * nr, r
    assert torch.equal(yio.to(torch.complex64), y32)


@pytest.mark.parametrize("nrhs", [1, 4, 8, 16])
def test_float_sums_stay_short(nrhs):
    """The c64 product's error against the plan's own FP64 product (2-lambda sphere,
    mean over 6 seeds) is that of sums over 32 lanes per row, 0.978e-7 with either 1
    or 16 right-hand sides, within 1%: fewer, longer float sums show here (one sum
    per lane of 16: 0.997e-7, 8 sums per row: 1.039e-7)."""
    from paper_1010_1456_amd import aim as A

    m = sphere_mesh(2.0, 0.3e9, nf=22, jitter_seed=1)
    plan = A.Plan([(m.verts, m.tris, 0.3e9)], cfie_alpha=0.6)
    err = 0.0
    for seed in range(6):
        g = torch.Generator(device="cuda").manual_seed(seed)
        x = torch.randn(nrhs, plan.n_total, dtype=torch.complex64, device="cuda", generator=g)
        y = plan.matvec(x, A.AIM_MIXED).to(torch.complex128)
        ref = plan.matvec(x.to(torch.complex128), A.AIM_FP64)
        err += float((y - ref).norm() / ref.norm()) / 6
    plan.close()
    assert err <= 0.988e-7


@pytest.mark.parametrize("nrhs", [1, 16])
def test_double_sums_stay_short(nrhs):
    """The interpolation and near product alone in FP64, on the fields the product leaves:
    rms against extended precision on the same fields, weights and near entries. Sums
    over 32 lanes per row have 1.52e-16 to 1.56e-16 here; half as many, twice as long,
    1.60e-16 to 1.70e-16."""
    from paper_1010_1456_amd import aim as A

    m = sphere_mesh(1.0, FREQ, nf=11, jitter_seed=1)
    k = wavenumber(FREQ)
    plan = A.Plan([(m.verts, m.tris, FREQ)], mixed=False)
    g = np.array(plan.info()["grid"][0])
    x = torch.randn(nrhs, plan.n_total, dtype=torch.complex128, device="cuda",
                    generator=torch.Generator(device="cuda").manual_seed(5))
    y = plan.matvec(x).cpu().numpy()
    phi = plan.product_stage(0, x, 6).cpu().numpy().reshape(nrhs, 4, -1)
    lam = plan.export(0, A.AIM_DATA_LAMBDA64).astype(np.longdouble)
    near = plan.export(0, A.AIM_DATA_NEAR64).astype(np.clongdouble)
    plan.close()
    h = A.host_plan(m.verts, m.tris, FREQ)
    u = np.stack(np.meshgrid(*[np.arange(3)] * 3, indexing="ij"), -1).reshape(-1, 3)
    node = h["anchors"][:, None] + u
    lin = (node[..., 0] * g[1] + node[..., 1]) * g[2] + node[..., 2]
    err = norm = np.longdouble(0)
    for r in range(min(nrhs, 2)):
        f = [(lam[:, q] * phi[r, q].astype(np.clongdouble)[lin]).sum(1) for q in range(4)]
        far = f[0] + f[1] + f[2] - np.longdouble(1.0 / (k * k)) * f[3]
        xr = x[r].cpu().numpy().astype(np.clongdouble)
        ref = 1j * np.longdouble(k * ETA0) * far + np.add.reduceat(near * xr[h["cols"]], h["rowptr"][:-1])
        err += (np.abs(y[r] - ref) ** 2).sum()
        norm += (np.abs(ref) ** 2).sum()
    assert np.sqrt(err / norm) <= 1.575e-16


@functools.lru_cache(maxsize=None)
def _larger(shape, order):
    from paper_1010_1456_amd import aim as A

    if shape == "sphere":  # 3 630 rows, no multiple of 8
        m, kw = sphere_mesh(1.0, FREQ, nf=11), {"cfie_alpha": 0.6}
    else:
        m, kw = plate_mesh(4.0, FREQ), {}  # 3 816 rows, planar
    return A.Plan([(m.verts, m.tris, FREQ)], order=order, near_radius_lambda=0.5, tune_rhs=17, **kw)


@pytest.mark.parametrize("nrhs", [6, 8, 9, 16, 17])
@pytest.mark.parametrize("shape,order", [("sphere", 1), ("sphere", 3), ("sphere", 5), ("plate", 2)])
def test_a_lane_each(shape, order, nrhs):
    """A lane per right-hand side, on meshes with rows enough for it, near rows and
    stencils in several stages: each product that of the right-hand side alone, with
    buffers that set-up left."""
    from paper_1010_1456_amd import aim as A

    plan = _larger(shape, order)
    held = plan.info()["device_bytes"]
    x = torch.from_numpy(random_current(plan.n_total, nrhs=nrhs, seed=nrhs)).cuda()
    for prec, dtype, tol in ((A.AIM_FP64, torch.complex128, 1e-12), (A.AIM_MIXED, torch.complex64, 2e-5)):
        xs = x.to(dtype)
        y = plan.matvec(xs, prec)
        assert plan.info()["device_bytes"] == held
        for r in range(nrhs):
            one = plan.matvec(xs[r], prec)
            assert torch.linalg.norm(y[r] - one) <= tol * torch.linalg.norm(one), r


@pytest.mark.parametrize("make,nrhs,multi,launches", [
    (lambda: plate_mesh(1.0, FREQ), 4, 0, 1),
    (lambda: plate_mesh(1.0, FREQ), 5, 0, 1),
    (lambda: plate_mesh(1.0, FREQ), 17, 0, 1),
    (lambda: plate_mesh(2.0, FREQ), 21, 0, 1),
    (lambda: plate_mesh(2.0, FREQ), 22, 1, 0),
    (lambda: plate_mesh(3.0, FREQ), 6, 1, 0),
    (lambda: sphere_mesh(0.5, FREQ, nf=6), 34, 0, 1),
    (lambda: sphere_mesh(0.5, FREQ, nf=6), 35, 1, 0),
    (lambda: sphere_mesh(1.0, FREQ, nf=11), 5, 0, 2),
    (lambda: sphere_mesh(1.0, FREQ, nf=11), 6, 1, 0),
])
def test_route(make, nrhs, multi, launches):
    """Few rows: rows (and a place in one launch) for each one or two of 3 or more right-hand
    sides, up to 20 480 rows together, or 36 864 of long lists per node (936 rows, and
    1 080 at fifth order); else groups of 4, from 6 on a lane each."""
    from torch.profiler import ProfilerActivity, profile

    from paper_1010_1456_amd import aim as A

    m = make()
    plan = A.Plan([(m.verts, m.tris, FREQ)], order=5 if nrhs > 30 else 3)
    x = torch.from_numpy(random_current(plan.n_total, nrhs=nrhs, seed=nrhs)).cuda()
    ref = plan.matvec(x[nrhs - 1], A.AIM_FP64)
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        y = plan.matvec(x, A.AIM_FP64)
        torch.cuda.synchronize()
    names = [e.name for e in prof.events()]
    assert sum("k_interp_multi<" in s for s in names) == multi
    assert sum("k_anterp_multi<" in s for s in names) == multi
    assert sum("k_interp_near<" in s for s in names) == launches
    assert torch.linalg.norm(y[nrhs - 1] - ref) <= 1e-12 * torch.linalg.norm(ref)
    plan.close()


@pytest.mark.parametrize("make,nrhs,fp64,kernel", [
    (lambda: plate_mesh(1.0, FREQ), 2, True, "2, false, 16"),
    (lambda: plate_mesh(2.0, FREQ), 3, True, "1, false, 16"),
    (lambda: sphere_mesh(0.7, FREQ, nf=8), 3, False, "1, false, 16"),  # 1 920 rows
    (lambda: plate_mesh(2.0, FREQ), 4, False, "2, false, 32"),
    (lambda: sphere_mesh(0.7, FREQ, nf=8), 4, False, "4, false, 16"),
    (lambda: sphere_mesh(0.85, FREQ, nf=9), 6, True, "2, false, 32"),
    (lambda: sphere_mesh(0.85, FREQ, nf=9), 11, True, "1, false, 16"),  # 2 430 rows
    (lambda: sphere_mesh(0.85, FREQ, nf=9), 13, True, "multi"),
    (lambda: sphere_mesh(1.0, FREQ, nf=11), 8, False, "4, false, 16"),  # 3 630 rows
    (lambda: sphere_mesh(1.0, FREQ, nf=11), 12, False, "4, false, 16"),
    (lambda: sphere_mesh(1.0, FREQ, nf=11), 8, True, "multi"),
    (lambda: sphere_mesh(1.0, FREQ, nf=11), 16, False, "multi"),
    (lambda: sphere_mesh(1.2, FREQ, nf=13), 12, False, "multi"),  # 5 070 rows
    (lambda: sphere_mesh(1.0, FREQ, nf=11), 1, True, "1, false, 32"),
    (lambda: plate_mesh(1.0, FREQ), 1, True, "1, false, 16"),
    (lambda: sphere_mesh(1.2, FREQ, nf=13), 1, True, "1, false, 16"),
])
def test_route_second_order(make, nrhs, fp64, kernel):
    """Second order keeps rows for each one or two up to 2 560 rows (28 672 together, 6 144 of 3 or 4
    right-hand sides), c64 full groups of 4 up to 49 152 rows together, and one
    right-hand side 32 lanes per row up to 4 096; set-up leaves the buffers of the route."""
    from torch.profiler import ProfilerActivity, profile

    from paper_1010_1456_amd import aim as A

    m = make()
    plan = A.Plan([(m.verts, m.tris, FREQ)], tune_rhs=nrhs)
    held = plan.info()["device_bytes"]
    prec = A.AIM_FP64 if fp64 else A.AIM_MIXED
    x = torch.from_numpy(random_current(plan.n_total, nrhs=nrhs, seed=nrhs)).cuda()
    x = x if fp64 else x.to(torch.complex64)
    few = plan.matvec(x[:max(nrhs - 1, 1)], prec)
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        y = plan.matvec(x, prec)
        torch.cuda.synchronize()
    assert plan.info()["device_bytes"] == held
    names = [e.name for e in prof.events() if "k_interp_" in e.name]
    arith = "double, double, double" if fp64 else "float, float, float"
    want = "k_interp_multi<" if kernel == "multi" else f"k_interp_near<{arith}, {kernel}>"
    assert len(names) == 1 and want in names[0], names
    tol = 1e-12 if fp64 else 2e-5
    assert torch.linalg.norm(y[0] - few[0]) <= tol * torch.linalg.norm(few[0])
    one = plan.matvec(x[nrhs - 1], prec)
    assert torch.linalg.norm(y[nrhs - 1] - one) <= tol * torch.linalg.norm(one)
    plan.close()
