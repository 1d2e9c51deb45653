"""State-dependent coefficients whose drift carries every node past its point,
on grids whose last tile has one point.

Measure and bar as in test_gpu_parity: max_i |gpu_i - oracle_i| /
max(|oracle_i|, 1) over the whole layer, <= 1e-10.
"""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import TOL64, lib, orc, rel_err, twin_half_width  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_x", [65, 129])
@pytest.mark.parametrize("kind", ["affine", "table"])
@pytest.mark.parametrize("K,L,cells", [(1, 1, 5.5), (3, 1, 40.0), (3, 7, 40.0), (3, 7, -40.0)])
def test_all_nodes_on_one_side(lib, orc, n_x, kind, K, L, cells):
    nt = 9
    wl = W.bidask_call_1d(n_x=n_x, n_t=nt, k=K, L=L, half_width=twin_half_width(0.2, 0.5, nt, n_x, 2.0))
    pb = wl.problem
    x = np.linspace(pb["x_min"], pb["x_max"], n_x)
    a = cells * (x[1] - x[0]) / (pb["T"] / nt)
    if kind == "affine":
        pb.update(vol_x=0.02 / (x[-1] - x[0]), vol=0.2 - 0.02 * x[0] / (x[-1] - x[0]), drift=a)
    else:
        pb["coef_tab"] = np.ascontiguousarray(np.stack([np.full(n_x, a), np.full(n_x, 0.2)])[None])
    iy, iz = wl.init_layers()
    print(f"[case] {kind} n_x {n_x} K {K} L {L} cells {cells}", flush=True)
    y, z, rc, _ = lib.solve(pb, iy, iz)
    assert rc == lib.BSDE_OK
    yo, zo, _ = orc.solve(pb, iy, iz)
    assert rel_err(y, yo) <= TOL64 and rel_err(z[0], zo[0]) <= TOL64
