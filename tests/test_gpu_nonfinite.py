"""Non-finite values in the initial layers reach the points whose nodes and
splines touch them, no others: zero weights are not multiplied with them.

One step from layers with an infinity (or a NaN) at some points, against the
same step from finite ones: away from those points (the nodes' reach and the
32 cells over which the truncated spline filter acts) the outputs keep every
bit.
"""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import TOL64, lib, rel_err, twin_half_width  # noqa: F401

pytestmark = pytest.mark.gpu

SPLINE = 34  # cells that a value's spline filter reaches, and one either side


def one_step(lib, pb, iy, iz):
    y, z, rc, _ = lib.solve(dict(pb, n_stop=pb["n_t"] - max(pb["k_y"], pb["k_z"])), iy, iz)
    assert rc in (lib.BSDE_OK, lib.BSDE_ENONFINITE, lib.BSDE_ENOCONV)
    return y, z


# one tile of 256 columns near both ends, two tiles, a short last one
@pytest.mark.parametrize("n1", [200, 256, 300])
@pytest.mark.parametrize("where", ["left", "right"])
@pytest.mark.parametrize("z_form", ["eq20", "yW"])
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_2d_end_column(lib, n1, where, z_form, value):
    n0 = 40
    wl = W.exchange_2d(n_x=n0, n_t=8)
    pb = dict(wl.problem, z_form=z_form)
    K = max(pb["k_y"], pb["k_z"])
    h = (pb["x_max"][1] - pb["x_min"][1]) / (n0 - 1)
    pb["n_x"] = [n0, n1]
    pb["x_max"] = [pb["x_max"][0], pb["x_min"][1] + h * (n1 - 1)]  # the cells keep their size
    rng = np.random.default_rng(7)
    iy, iz = rng.normal(size=(K, n0, n1)), rng.normal(size=(K, 2, n0, n1))
    y, z = one_step(lib, pb, iy.reshape(K, -1), iz.reshape(K, 2, -1))
    col = 0 if where == "left" else n1 - 1
    iy[:, :, col] = value
    print(f"[case] n1 {n1} {where} {z_form} {value}", flush=True)
    yb, zb = one_step(lib, pb, iy.reshape(K, -1), iz.reshape(K, 2, -1))
    reach = lib.bsde_problem_info(pb)["node_reach"] + SPLINE
    far = np.abs(np.arange(n1) - col) > reach
    assert far.sum() > 40
    pick = lambda a: np.asarray(a).reshape(-1, n0, n1)[:, :, far]
    assert np.isfinite(pick(yb)).all() and np.isfinite(pick(zb)).all()
    assert np.array_equal(pick(yb), pick(y)) and np.array_equal(pick(zb), pick(z))


# every node of every point beyond the end (a drift of more than the grid): the
# outputs depend on the end values alone, whatever is inside
@pytest.mark.parametrize("side", [-1.0, 1.0])
@pytest.mark.parametrize("kind", ["const", "located", "exact", "2d"])
@pytest.mark.parametrize("at", [2, 35, 67])
def test_nodes_beyond_the_end_take_its_value(lib, side, kind, at):
    nt, n = 9, 70
    if kind == "2d":
        pb = dict(W.exchange_2d(n_x=n, n_t=nt).problem)
        dx = (pb["x_max"][0] - pb["x_min"][0]) / (n - 1)
        pb["drift"] = [side * 200 * dx / (pb["T"] / nt), pb["drift"][1]]
        K, shape = max(pb["k_y"], pb["k_z"]), (n, n)
    else:
        wl = W.bs_call_1d(n_x=n, n_t=nt, k=3, L=8, half_width=twin_half_width(0.2, 0.33, nt, n, 3.0))
        pb = dict(wl.problem)
        dx = (pb["x_max"] - pb["x_min"]) / (n - 1)
        pb["drift"] = side * 200 * dx / (pb["T"] / nt)
        if kind == "located":
            pb["vol_x"] = 1e-3
        if kind == "exact":
            pb["quad"] = "exact"
        K, shape = 3, (n,)
    rng = np.random.default_rng(11)
    iy = rng.normal(size=(K,) + shape)
    iz = rng.normal(size=(K, len(shape)) + shape)
    flat = lambda a, d: np.ascontiguousarray(a.reshape(K, -1) if d == 1 else a.reshape(K, len(shape), -1))
    y, z = one_step(lib, pb, flat(iy, 1), flat(iz, 2))
    # along axis 0, a non-finite point inside the grid; the implicit equation
    # starts from the point's own y, so that point is left out
    iy[:, at] = np.nan
    print(f"[case] {kind} side {side} at {at}", flush=True)
    yb, zb = one_step(lib, pb, flat(iy, 1), flat(iz, 2))
    y, yb = np.asarray(y).reshape(shape), np.asarray(yb).reshape(shape)
    z, zb = np.asarray(z).reshape((-1,) + shape), np.asarray(zb).reshape((-1,) + shape)
    # (located nodes take an end's value by their weights where all records are
    # finite and by itself where not: the same up to rounding)
    keep = np.arange(n) != at
    assert np.isfinite(yb[keep]).all() and np.isfinite(zb).all()
    assert rel_err(yb[keep], y[keep]) <= TOL64 and rel_err(zb, z) <= TOL64
