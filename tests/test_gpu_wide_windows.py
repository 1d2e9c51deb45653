"""Wide node windows on grids either side of the line between the fused sweep and
the direct kernel: the plan's choice, and the same results from the autotuner's.

Measure and bar as in test_gpu_parity: max_i |gpu_i - oracle_i| /
max(|oracle_i|, 1) over the whole layer, <= 1e-10.
"""
import pytest

import workloads as W
from test_gpu_parity import TOL64, batched_solve, lib, orc, rel_err, twin_half_width  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_x", [16385, 65537])
@pytest.mark.parametrize("autotune", [False, True])
def test_wide_windows(lib, orc, n_x, autotune):
    # ratio 105 at K = 4, L = 16: only 64-point tiles fit LDS; few steps, as the
    # scheme is unstable there
    nt = 6
    wl = W.bidask_call_1d(n_x=n_x, n_t=nt, k=4, L=16, half_width=twin_half_width(0.2, 0.5, nt, n_x, 105.0))
    print(f"[case] n_x {n_x} autotune {autotune}", flush=True)
    rc, _, outs, rep = batched_solve(lib, [wl], autotune=autotune)
    assert rc == lib.BSDE_OK
    iy, iz = wl.init_layers()
    yo, zo, _ = orc.solve(wl.problem, iy, iz)
    y, z = outs[0]
    assert rel_err(y, yo) <= TOL64 and rel_err(z, zo[0]) <= TOL64
    if autotune:  # the fused shape that fits, and both direct ones
        assert rep["candidates"] == 3
