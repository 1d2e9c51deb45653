"""The fused 1-D sweep at the sizes where its tiles, node classes, windows and
end handling can go wrong, in every shape that the plan picks by itself.

Measure and bars as in test_gpu_parity: max_i |gpu_i - oracle_i| /
max(|oracle_i|, 1) over the whole layer, <= 1e-10 in FP64, <= 1e-6 in the FP32
form (the oracle works in double precision; one step errs by a few units in
the last place per node sum, a few dozen steps by well under the bar).
"""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import TOL32, TOL64, lib, orc, rel_err, twin_half_width  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES64 = ["fused:1:8:1", "fused:2:8:1", "fused:4:8:1", "fused:4:4:4"]
SHAPES32 = ["fused:1:1:2", "fused:1:1:4", "fused:1:1:8", "fused:1:1:16"]


def solve(lib, pb, iy, iz):
    y, z, rc, _ = lib.solve(pb, iy, iz)
    assert rc == lib.BSDE_OK
    return y, z[0]


# 64-point tiles and their remainders, one period of the reflected
# continuation and less than one, both ends inside one wavefront's reach
@pytest.mark.parametrize("n_x", [4, 33, 64, 65, 127, 1023, 2049])
@pytest.mark.parametrize("K,L", [(1, 1), (2, 7), (3, 12), (6, 16)])
def test_shapes_agree_and_match_oracle(lib, orc, monkeypatch, n_x, K, L):
    wl = W.bidask_call_1d(n_x=n_x, n_t=10, k=K, L=L, half_width=twin_half_width(0.2, 0.5, 10, n_x, 9.0))
    iy, iz = wl.init_layers()
    yo, zo, _ = orc.solve(wl.problem, iy, iz)
    first = None
    for spec in SHAPES64:
        print(f"[case] {spec} n_x {n_x} K {K} L {L}", flush=True)
        monkeypatch.setenv("BSDE_SWEEP", spec)
        y, z = solve(lib, wl.problem, iy, iz)
        assert rel_err(y, yo) <= TOL64 and rel_err(z, zo[0]) <= TOL64
        if first is None:
            first = (y, z)
        # the same sums in every shape
        assert np.array_equal(y, first[0]) and np.array_equal(z, first[1])


@pytest.mark.parametrize("n_x", [65, 1025, 8193 + 511])
@pytest.mark.parametrize("K", [1, 4, 5])
def test_fp32_shapes_agree_and_match_oracle(lib, orc, monkeypatch, n_x, K):
    wl = W.bidask_call_1d(n_x=n_x, n_t=10, k=K, L=16, half_width=twin_half_width(0.2, 0.5, 10, n_x, 9.0))
    pb = dict(wl.problem, prec="fp32_comp")
    iy, iz = wl.init_layers()
    yo, zo, _ = orc.solve(pb, iy, iz)
    first = None
    for spec in SHAPES32:
        print(f"[case] {spec} n_x {n_x} K {K}", flush=True)
        monkeypatch.setenv("BSDE_SWEEP", spec)
        y, z = solve(lib, pb, iy, iz)
        assert rel_err(y, yo) <= TOL32 and rel_err(z, zo[0]) <= TOL32
        if first is None:
            first = (y, z)
        assert np.array_equal(y, first[0]) and np.array_equal(z, first[1])


# wide windows (L = 32, 64), every driver, a linear driver with a constant term
@pytest.mark.parametrize("case", ["bs32", "bs64", "cubic", "exp", "constant"])
def test_drivers_and_wide_windows(lib, orc, case):
    if case == "bs32":
        wl = W.bs_call_1d(n_x=3001, n_t=12, k=6, L=32, half_width=twin_half_width(0.2, 0.33, 12, 3001))
    elif case == "bs64":
        wl = W.bs_call_1d(n_x=2003, n_t=12, k=4, L=64, half_width=twin_half_width(0.2, 0.33, 12, 2003, 10.0))
    elif case == "cubic":
        wl = W.paper_example1(4, 16, 700)
    elif case == "exp":
        wl = W.paper_example2(4, 16, 700)
    else:
        wl = W.bs_call_1d(n_x=1500, n_t=12, k=3, L=16, half_width=twin_half_width(0.2, 0.33, 12, 1500, 8.0))
        p = list(wl.problem["p"])
        p[3] = 0.7
        wl.problem["p"] = p
    iy, iz = wl.init_layers()
    y, z = solve(lib, wl.problem, iy, iz)
    yo, zo, _ = orc.solve(wl.problem, iy, iz)
    assert rel_err(y, yo) <= TOL64 and rel_err(z, zo[0]) <= TOL64
