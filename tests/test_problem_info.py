"""The node reach that a problem reports: the scheme's own, whichever kernel and
windows serve it (host only)."""
import pytest

import paper_1909_13560_amd as lib
import workloads as W


@pytest.mark.parametrize("prec", ["fp64", "fp32_comp"])
@pytest.mark.parametrize("make,reach", [
    (lambda: W.exchange_2d(n_x=33, n_t=6), 8),
    (lambda: W.basket_2d(n_x=65, n_t=12), 24),
    (lambda: W.ou_linear_1d(n_x=801, n_t=32), 89),
    (lambda: W.tabulated(W.ou_linear_1d(n_x=801, n_t=32), True), 82),
])
def test_node_reach(make, reach, prec):
    assert lib.bsde_problem_info(dict(make().problem, prec=prec))["node_reach"] == reach
