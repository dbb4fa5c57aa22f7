"""How the planner cuts circuits into passes (no GPU needed)."""
import os

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


# Priced planning never returns a plan that it prices above the default one.
@pytest.mark.parametrize("mode", ["profiled", "learned"])
@pytest.mark.parametrize("n", [13, 16, 18, 19, 20])
@pytest.mark.parametrize("prec", [0, 1])
def test_priced_plan_against_the_default(prec, n, mode):
    models = os.path.join(os.path.dirname(q.__file__), "models")
    if mode == "profiled":
        kw = {"mode": q.PLAN_PROFILED, "profile": q.Profile.load(os.path.join(models, "corpus_profile.bin"))}
    else:
        kw = {"mode": q.PLAN_LEARNED, "model": q.CostModel.load(os.path.join(models, "cost_mlp.bin"))}
    for seed in range(3):
        for c in (W.haar_blocks(seed, n, 40), W.random_mixed(seed, n, 80, max_dense_k=5), W.random_mix_layers(seed, n, 10)):
            best = q.Plan(n, c.gates, precision=prec, **kw).stats()["predicted_s"]
            default = q.Plan(n, c.gates, precision=prec).predict(**kw)
            assert best <= default * (1 + 1e-12), (seed, c.name)
