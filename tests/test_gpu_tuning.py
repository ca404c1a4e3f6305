"""What set-up times with a hint of several right-hand sides: the projection gather
that up to five take, with its three widths, and the projection fused with the z pass
that one takes, are timed as such (not on a launch that has no such variants, whose
noise would then choose them)."""

import pytest

from workloads import sphere_mesh

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

FREQ = 0.3e9


@pytest.mark.parametrize("hint", [0, 5, 6, 16])
def test_timed_kernels(hint):
    from torch.profiler import ProfilerActivity, profile

    from paper_1010_1456_amd import aim as A

    m = sphere_mesh(0.4, FREQ, nf=3)
    A.Plan([(m.verts, m.tris, FREQ)]).close()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        plan = A.Plan([(m.verts, m.tris, FREQ)], fft_min_pad=192, tune_rhs=hint)
        torch.cuda.synchronize()
    names = [e.name for e in prof.events()]
    for arith in ("double", "float"):
        # 3 widths, and the two-launch form of the z pass, 4 repetitions each
        assert sum(f"k_anterp_gather<{arith}" in s for s in names) == 16, arith
        assert sum(f"k_anterp_fftz<{arith}" in s for s in names) == 4, arith
    plan.close()
