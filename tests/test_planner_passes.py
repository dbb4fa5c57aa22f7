"""How the planner cuts circuits into passes (no GPU needed)."""
import pytest

import paper_2410_09326_amd as q
from workloads import circuits as W


# A register tile pass stages no coefficients in LDS, so the LDS beside the
# tile must not end it.
@pytest.mark.parametrize("n,depth,up", [(13, 21, 7), (13, 128, 7), (12, 140, 0), (10, 300, 0)])
@pytest.mark.parametrize("prec", [0, 1])
def test_whole_state_tile_is_one_pass(n, depth, up, prec):
    c = W.param_sweep_batch(seed=depth, count=1, nmin=n, nmax=n, dmin=depth, dmax=depth)[0]
    p = q.Plan(n, c.gates, precision=prec, tile_upper=up)
    assert [x["type"] for x in p.passes()] == [0]


# Four times the operations in one pass: about four times the planning (16
# times if every new register set looked at the whole pass again).
@pytest.mark.parametrize("n,up", [(12, 0), (13, 7)])
@pytest.mark.parametrize("prec", [0, 1])
def test_planning_is_linear_in_a_pass(n, up, prec):
    def seconds(layers):
        c = W.layered_u3_cx(1, n=n, depth=layers, swap_frac=0.0)
        return min(q.Plan(n, c.gates, precision=prec, tile_upper=up).stats()["plan_seconds"] for _ in range(3))
    assert seconds(6000) <= 9 * seconds(1500)
