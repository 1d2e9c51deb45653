"""State-dependent coefficients on grids whose plan takes 256-point tiles: tile
remainders, few and many nodes, a batch against its instances alone (64-point
tiles, the same bits), and the autotuner's choice.

Measure and bar as in test_gpu_parity: max_i |gpu_i - oracle_i| /
max(|oracle_i|, 1) over the whole layer, <= 1e-10.
"""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import TOL64, batched_solve, lib, orc, rel_err, twin_half_width  # noqa: F401

pytestmark = pytest.mark.gpu


def affine(n_x, nt, K, L, R):
    wl = W.bidask_call_1d(n_x=n_x, n_t=nt, k=K, L=L, half_width=twin_half_width(0.2, 0.5, nt, n_x, R))
    pb = wl.problem
    pb["vol_x"] = 0.04 / (pb["x_max"] - pb["x_min"])
    pb["vol"] = 0.2 - pb["vol_x"] * pb["x_max"]
    return wl


@pytest.mark.parametrize("n_x", [131072, 131073, 131071])
@pytest.mark.parametrize("K,L", [(1, 1), (1, 4), (2, 8), (3, 16)])
def test_large_grid(lib, orc, n_x, K, L):
    wl = affine(n_x, 5, K, L, 9.0)
    iy, iz = wl.init_layers()
    print(f"[case] n_x {n_x} K {K} L {L}", flush=True)
    y, z, rc, _ = lib.solve(wl.problem, iy, iz)
    assert rc == lib.BSDE_OK
    yo, zo, _ = orc.solve(wl.problem, iy, iz)
    assert rel_err(y, yo) <= TOL64 and rel_err(z[0], zo[0]) <= TOL64


@pytest.mark.parametrize("autotune", [False, True])
def test_batch_gives_the_bits_of_its_instances(lib, autotune):
    wls = [affine(n, 7, 2, 8, 6.0 + i % 5) for i, n in enumerate([2001, 500, 64, 65, 1023] * 30)]
    rc, _, outs, rep = batched_solve(lib, wls, autotune=autotune)
    assert rc == lib.BSDE_OK
    if autotune:
        print(f"[case] {rep}", flush=True)
        assert rep["path"] == 3 and rep["candidates"] >= 2
    for i in range(0, len(wls), 7):
        iy, iz = wls[i].init_layers()
        y, z, _, _ = lib.solve(wls[i].problem, iy, iz)
        assert np.array_equal(outs[i][0], y) and np.array_equal(outs[i][1], z[0])
