"""Exact expectations in batches whose plan takes one wavefront group, or the
chunked sweep.

Measure and bar as in test_gpu_parity: max_i |gpu_i - oracle_i| /
max(|oracle_i|, 1) over the whole layer, <= 1e-10.
"""
import types

import numpy as np
import pytest
import torch

import workloads as W
from test_gpu_parity import TOL64, batched_solve, lib, orc, rel_err, twin_half_width  # noqa: F401

pytestmark = pytest.mark.gpu


def exact_call(n_x, K, R, nt):
    wl = W.bs_call_1d(n_x=n_x, n_t=nt, k=K, L=8, half_width=twin_half_width(0.2, 0.33, nt, n_x, R))
    pb = dict(wl.problem, quad="exact")
    # (the price itself would overflow on an interval this wide)
    x = np.arange(n_x) * 0.003
    iy = np.stack([np.sin(x + 0.1 * r) + 1.5 for r in range(K)])
    iz = np.stack([np.cos(x + 0.1 * r) * 0.2 for r in range(K)])[:, None]
    return types.SimpleNamespace(problem=pb, init_layers=lambda: (iy, iz))


# batches of 4096 tiles and more (the group's tiles decide): one group on B-spline
# coefficients; the chunked sweep (narrow bands, one block a CU); instances of
# uneven lengths with tile remainders of 1, of all but 1, and none
@pytest.mark.parametrize("K,R,path", [(4, 8.0, "one group"), (2, 8.0, "one group"), (2, 2.0, "chunked"),
                                      (1, 4.0, "chunked"), (2, 45.0, "chunked")])
def test_large_batch(lib, orc, K, R, path):
    wls = [exact_call(4096 + (i % 3) - 1, K, R, K + 2 + i % 3) for i in range(70)]
    print(f"[case] K {K} R {R} {path}", flush=True)
    rc, _, outs, _ = batched_solve(lib, wls)
    assert rc == lib.BSDE_OK
    for i in (0, 1, 2, 35, 69):
        iy, iz = wls[i].init_layers()
        yo, zo, _ = orc.solve(wls[i].problem, iy, iz)
        assert rel_err(outs[i][0], yo) <= TOL64 and rel_err(outs[i][1], zo[0]) <= TOL64
    # which kernel that was: the chunked one builds its spline in launches of its own
    plan = lib.bsde_plan([w.problem for w in wls])
    ws = lib.workspace(plan)
    ios = []
    for w in wls:
        iy, iz = w.init_layers()
        ios.append((torch.as_tensor(iy, device="cuda"), torch.as_tensor(iz[:, 0], device="cuda").contiguous(),
                    torch.empty(iy.shape[1], dtype=torch.float64, device="cuda"),
                    torch.empty(iy.shape[1], dtype=torch.float64, device="cuda")))
    kt = lib.bsde_profile_kernels(plan, ws, ios)
    assert kt["path"] == 4 and kt["node_groups"] == 1
    assert (kt["spline_launches"] > 0) == (path == "chunked")
