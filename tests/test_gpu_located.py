"""State-dependent coefficients in the fused sweep: window bounds, tile
remainders and the clamped ends, for affine and tabulated coefficients.

Measure and bar as in test_gpu_parity: max_i |gpu_i - oracle_i| /
max(|oracle_i|, 1) over the whole layer, <= 1e-10.
"""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import TOL64, lib, orc, rel_err, twin_half_width  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_x", [4, 64, 65, 500, 1023])
@pytest.mark.parametrize("kind", ["affine", "table", "steps"])
@pytest.mark.parametrize("K,L", [(1, 1), (3, 16), (6, 7)])
def test_located_nodes(lib, orc, n_x, kind, K, L):
    nt = 9
    wl = W.bidask_call_1d(n_x=n_x, n_t=nt, k=K, L=L, half_width=twin_half_width(0.2, 0.5, nt, n_x, 6.0))
    pb = wl.problem
    x = np.linspace(pb["x_min"], pb["x_max"], n_x)
    u = (x - x[0]) / (x[-1] - x[0])
    dx = x[1] - x[0]
    if kind == "affine":  # volatility doubles over the grid, drift changes sign
        pb.update(vol=0.1 - 0.1 * x[0] / (x[-1] - x[0]), vol_x=0.1 / (x[-1] - x[0]),
                  drift=0.0, drift_x=0.0)
    else:
        rows = nt if kind == "steps" else 1
        s = np.arange(rows)[:, None]
        a = 20 * dx / (pb["T"] / nt) * np.sin(6 * u[None] + s)  # up to 20 cells a step
        b = 0.2 * (1.0 + 0.4 * np.cos(9 * u[None] - 0.3 * s))
        pb["coef_tab"] = np.ascontiguousarray(np.stack([a, b], axis=1))
    iy, iz = wl.init_layers()
    print(f"[case] {kind} n_x {n_x} K {K} L {L}", flush=True)
    y, z, rc, _ = lib.solve(pb, iy, iz)
    assert rc == lib.BSDE_OK
    yo, zo, _ = orc.solve(pb, iy, iz)
    assert rel_err(y, yo) <= TOL64 and rel_err(z[0], zo[0]) <= TOL64
