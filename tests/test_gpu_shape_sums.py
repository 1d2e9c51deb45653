"""Every shape of the FP64 fused sweep adds a point's nodes in the same order,
also where a block has one or two node groups and its lists are long.

Measure and bar as in test_gpu_parity: max_i |gpu_i - oracle_i| /
max(|oracle_i|, 1) over the whole layer, <= 1e-10.
"""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import TOL64, lib, orc, rel_err, twin_half_width  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = ["fused:1:8:1", "fused:4:4:4", "fused:1:1", "fused:1:2", "fused:2:1", "fused:2:2", "fused:4:1",
          "fused:4:2"]


# K L from less than a node per class to the most; (6, 19..21), (5, 25) and
# (3, 42) have more than 64 nodes in half of the classes, on average fewer
@pytest.mark.parametrize("K,L", [(1, 3), (4, 16), (6, 19), (6, 20), (6, 21), (5, 25), (3, 42), (6, 64)])
def test_every_shape_gives_the_same_sums(lib, orc, monkeypatch, K, L):
    n_x = 1300
    wl = W.bidask_call_1d(n_x=n_x, n_t=10, k=K, L=L, half_width=twin_half_width(0.2, 0.5, 10, n_x, 6.0))
    iy, iz = wl.init_layers()
    yo, zo, _ = orc.solve(wl.problem, iy, iz)
    first = None
    for spec in SHAPES:
        print(f"[case] {spec} K {K} L {L}", flush=True)
        monkeypatch.setenv("BSDE_SWEEP", spec)
        y, z, rc, _ = lib.solve(wl.problem, iy, iz)
        assert rc == lib.BSDE_OK
        assert rel_err(y, yo) <= TOL64 and rel_err(z[0], zo[0]) <= TOL64
        if first is None:
            first = (y, z)
        assert np.array_equal(y, first[0]) and np.array_equal(z, first[1])
