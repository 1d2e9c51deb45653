"""The 2-D sweep on value and derivative planes (FP32 spline, bicubic) on both
sides of the tile counts where its staging changes.

FP64: max_i |gpu_i - oracle_i| / max(|oracle_i|, 1) over the whole layer
<= 1e-10; FP32 form: the parity tests' FP32 bound.  The bicubic runs in FP64
only: its fourth-order differences amplify the FP32 form's rounding on axes of
few points (512 x 9: 1.2e-6, whichever kernel takes the step).
"""
import pytest

import workloads as W
from test_gpu_parity import TOL32, TOL64, lib, orc, rel_err  # noqa: F401

pytestmark = pytest.mark.gpu


# rows: 256 and 512 one-column tiles and one more; columns: less than a
# wavefront's 128, one column into the second wavefront, two 512-column tiles
# with 3 columns in the last, a node spread whose two windows take over 64 KB
@pytest.mark.parametrize("n0,n1", [(256, 40), (257, 129), (512, 9), (513, 40), (7, 127), (6, 515),
                                   (129, 640), (33, 760)])
@pytest.mark.parametrize("prec,interp", [("fp32_comp", "spline"), ("fp64", "bicubic_fd")])
def test_tile_counts(lib, orc, n0, n1, prec, interp):
    wl = W.exchange_2d(n_x=max(n0, n1), n_t=6, k=2, L=5, rho=0.4)
    pb = wl.problem
    pb.update(n_x=[n0, n1], interp=interp)
    iy, iz = wl.init_layers()
    print(f"[case] {n0} x {n1} {prec} {interp}", flush=True)
    y, z, rc, _ = lib.solve(dict(pb, prec=prec), iy, iz)
    assert rc == lib.BSDE_OK
    yo, zo, _ = orc.solve(pb, iy, iz)
    tol = TOL32 if prec == "fp32_comp" else TOL64
    assert rel_err(y, yo) <= tol
    for c in range(2):
        assert rel_err(z[c], zo[c]) <= tol
