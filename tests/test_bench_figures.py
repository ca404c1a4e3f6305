"""The benchmark's per-step figures where one kernel runs the y, x and inverse y passes
plane by plane: kernels are attributed to the steps they run, the step that carries the
three passes gets their bytes (unpadded planes in and out), and a scatterer without an x
pass of its own adds no operations to one (CPU)."""

import numpy as np
import pytest

import bench

INFO = dict(nmesh=2, order=2, n=[100, 50], nnz=[900, 300], grid=[(21, 21, 21), (11, 13, 3)],
            pad=[(42, 42, 42), (21, 25, 5)], occ_nodes=[2000, 143], occ_lines=[400, 143],
            planar_z=[-1, 1], cfie_alpha=[0.6, None], fused_projection=[(False, True), (False, False)],
            xy_groups=[(1, 1), (1, 1)])
A, Z, Y = "k_anterp_gather<float, double>", "k_fft_contig<float, false, true, PlanC<6, 7, 1> >", \
    "k_fft_strided<float, false, true, PlanC<6, 7, 1>, 128>"
X, YI, ZI = "k_fft_mid<float, PlanC<6, 7, 1>, false, 128, true>", Y.replace("false", "true"), \
    Z.replace("false", "true")
ZP, P = "k_fft_zplane<float, false, true, PlanC<6, 7, 1> >", "k_fft_plane<float, PlanC<6, 7, 1>, true>"
I = "k_interp_near<float, double, double, 1, true, 16>"


@pytest.mark.parametrize("names,planar,stages", [
    ([A, Z, Y, X, YI, ZI, I], False, {0: A, 1: Z, 2: Y, 3: X, 4: YI, 5: ZI, 6: I}),
    (["k_anterp_fftz<float>", Y, X, YI, ZI, I], False,
     {0: "k_anterp_fftz<float>", 2: Y, 3: X, 4: YI, 5: ZI, 6: I}),
    (["k_transpose_x<float, double>", "k_anterp_multi<float, 16>", ZP, P, ZP.replace("false", "true"),
      "k_interp_multi<float, double, 16, true>"], False,
     {0: "k_anterp_multi<float, 16>", 1: ZP, 2: P, 5: ZP.replace("false", "true"),
      6: "k_interp_multi<float, double, 16, true>"}),
    ([A, Z, X, ZI, I], True, {0: A, 2: Z, 3: X, 4: ZI, 6: I}),
    ([A, P, I], True, {0: A, 2: P, 6: I}),
])
def test_kernel_stages(names, planar, stages):
    assert bench.kernel_stages(names, planar) == stages


@pytest.mark.parametrize("mesh", [0, 1])
def test_plane_by_plane_bytes(mesh):
    args = (INFO, mesh, 3, 8, 4, 16, 16, 1)
    sep, pl = bench.stage_bytes(*args), bench.stage_bytes(*args, planes=True)
    px, py, pz = INFO["pad"][mesh]
    h = (px // 2 + 1) * (py // 2 + 1) * (1 if mesh else pz // 2 + 1)
    moved = 12 * (11 * 13 if mesh else 400 * 42)
    assert pl[2] == 8 * (2 * moved + h) and pl[3] == pl[4] == 0.0
    assert np.array_equal(np.delete(pl, [2, 3, 4]), np.delete(sep, [2, 3, 4]))
    assert pl[2] < sep[2] + sep[3] + sep[4]


def test_x_pass_operations_of_scatterers_that_have_one():
    both = bench.x_pass_flops(INFO, 3, [False, False])
    assert both == bench.x_pass_flops(INFO, 3, [True, False]) + bench.x_pass_flops(INFO, 3, [False, True])
    assert bench.x_pass_flops(INFO, 3, [True, True]) == 0.0
    assert bench.x_pass_alu(INFO, 3, 0.1, [True, True]) is None


def test_traffic_digest_covers_the_tables_a_product_reads():
    for name in ("node_tables.hip", "near_pattern.hip", "scan.h", "fft_plane.h", "multi_rhs.h"):
        assert name not in bench.MATVEC_SOURCES_EXCLUDED
