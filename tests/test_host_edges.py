"""The host planner's RWG table on meshes whose vertices hold more edges than its
small sort takes (a fan, the hub numbered first or last) and with shuffled
triangles, against the oracle (CPU)."""

import numpy as np
import pytest

from oracle.rwg import build_rwg
from paper_1010_1456_amd import aim as A


@pytest.mark.parametrize("hub_first", [False, True])
@pytest.mark.parametrize("n", [3, 31, 33, 200])
def test_fan(n, hub_first):
    ang = np.linspace(0.0, 2.0 * np.pi, n, endpoint=False)
    v = np.concatenate([np.stack([np.cos(ang), np.sin(ang), 0.1 * np.sin(5 * ang)], 1),
                        [[0.0, 0.0, 0.2]]])
    t = np.array([[n, i, (i + 1) % n] for i in range(n)])
    if hub_first:
        new = np.roll(np.arange(n + 1), -1)  # vertex i -> i + 1, the hub -> 0
        w = np.empty_like(v)
        w[new] = v
        v, t = w, new[t]
    t = t[np.random.default_rng(n).permutation(n)].astype(np.int32)
    r = build_rwg(v, t)
    ref = np.stack([r.edge[:, 0], r.edge[:, 1], r.tplus, r.tminus, r.vplus, r.vminus], 1)
    assert np.array_equal(A.host_plan(v, t, 0.3e9)["rwg"], ref)
