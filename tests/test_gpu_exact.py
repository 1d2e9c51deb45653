"""Exact Gaussian expectations on B-spline coefficients at the sizes where the
64-point tiles, the 4-tap steps and the end corrections can go wrong.

Measure and bar as in test_gpu_parity: max_i |gpu_i - oracle_i| /
max(|oracle_i|, 1) over the whole layer, <= 1e-10.
"""
import pytest

import workloads as W
from test_gpu_parity import TOL64, lib, orc, rel_err, twin_half_width  # noqa: F401

pytestmark = pytest.mark.gpu


# grids inside one band's reach (both corrections at every point), tile
# remainders of 1 and 63, several tiles; drifts that move the band off its centre
@pytest.mark.parametrize("n_x", [4, 64, 65, 127, 700, 2049])
@pytest.mark.parametrize("K,R,drift,z_form", [(1, 3.0, None, "yW"), (2, 9.0, None, "eq20"),
                                              (6, 16.0, None, "eq20"), (3, 6.0, 40.0, "eq20"),
                                              (3, 6.0, -40.0, "eq20")])
def test_exact_tiles_and_ends(lib, orc, n_x, K, R, drift, z_form):
    wl = W.bs_call_1d(n_x=n_x, n_t=10, k=K, L=8, half_width=twin_half_width(0.2, 0.33, 10, n_x, R))
    pb = wl.problem
    pb.update(quad="exact", z_form=z_form)
    if drift is not None:  # cells per step
        dx = (pb["x_max"] - pb["x_min"]) / (n_x - 1)
        pb["drift"] = drift * dx / (pb["T"] / pb["n_t"])
    p = list(pb["p"])
    p[3] = 0.4  # the driver's constant term
    pb["p"] = p
    iy, iz = wl.init_layers()
    print(f"[case] n_x {n_x} K {K} R {R} drift {drift}", flush=True)
    y, z, rc, _ = lib.solve(pb, iy, iz)
    assert rc == lib.BSDE_OK
    yo, zo, _ = orc.solve(pb, iy, iz)
    assert rel_err(y, yo) <= TOL64 and rel_err(z[0], zo[0]) <= TOL64
