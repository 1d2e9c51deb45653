"""The 2-D sweep on B-spline coefficients (FP64, natural spline) where its
tiles, node rows and end corrections can go wrong.

Measure and bar as in test_gpu_parity: max_i |gpu_i - oracle_i| /
max(|oracle_i|, 1) over the whole layer, <= 1e-10.
"""
import pytest

import workloads as W
from test_gpu_parity import TOL64, lib, orc, rel_err  # noqa: F401

pytestmark = pytest.mark.gpu


# axis lengths: shorter than the filter's reach, both ends within one node's
# reach, the 256-column tile and its remainders, two tiles
@pytest.mark.parametrize("n0,n1", [(4, 5), (5, 40), (33, 255), (21, 256), (40, 257), (9, 515)])
@pytest.mark.parametrize("z_form", ["eq20", "yW"])
def test_tiles_and_ends(lib, orc, n0, n1, z_form):
    wl = W.exchange_2d(n_x=max(n0, n1), n_t=6, k=2, L=5, rho=0.4)
    pb = wl.problem
    pb.update(n_x=[n0, n1], z_form=z_form)
    pb["p"] = list(pb["p"][:3]) + [0.3]  # the driver's constant term
    iy, iz = wl.init_layers()
    print(f"[case] {n0} x {n1} z_form {z_form}", flush=True)
    y, z, rc, _ = lib.solve(pb, iy, iz)
    assert rc == lib.BSDE_OK
    yo, zo, _ = orc.solve(pb, iy, iz)
    assert rel_err(y, yo) <= TOL64
    for c in range(2):
        assert rel_err(z[c], zo[c]) <= TOL64
