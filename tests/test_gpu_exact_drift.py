"""Exact expectations whose whole band lies to one side of the point, on grids
whose last tile has one point.

Measure and bar as in test_gpu_parity: max_i |gpu_i - oracle_i| /
max(|oracle_i|, 1) over the whole layer, <= 1e-10.
"""
import pytest

import workloads as W
from test_gpu_parity import TOL64, lib, orc, rel_err, twin_half_width  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_x", [64, 65, 129])
@pytest.mark.parametrize("K,drift", [(1, -60.0), (3, -60.0), (3, -130.0), (1, 60.0), (3, 130.0)])
def test_band_beside_the_tile(lib, orc, n_x, K, drift):
    wl = W.bs_call_1d(n_x=n_x, n_t=10, k=K, L=8, half_width=twin_half_width(0.2, 0.33, 10, n_x, 3.0))
    pb = wl.problem
    dx = (pb["x_max"] - pb["x_min"]) / (n_x - 1)
    pb.update(quad="exact", drift=drift * dx / (pb["T"] / pb["n_t"]))  # cells per step
    iy, iz = wl.init_layers()
    print(f"[case] n_x {n_x} K {K} drift {drift}", flush=True)
    y, z, rc, _ = lib.solve(pb, iy, iz)
    assert rc == lib.BSDE_OK
    yo, zo, _ = orc.solve(pb, iy, iz)
    assert rel_err(y, yo) <= TOL64 and rel_err(z[0], zo[0]) <= TOL64
