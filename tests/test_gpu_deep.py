"""Deep circuits on states that one register tile holds (10-13 qubits) or
whose busy qubits fit one: every operation runs in one pass, with nothing
stored in between, so chains of 2x2s get long.  Against the oracle."""
import functools

import numpy as np
import pytest

from oracle import oracle as orc
from workloads import circuits as W

pytestmark = pytest.mark.gpu

GATES = {"h": ("h", ()), "rx": ("rx", (np.pi / 2,)), "ry": ("ry", (1.1,))}


def layers_of(kind, params, busy, layers):
    gates = []
    for i in range(layers):
        gates += [W.Gate(kind, (b,), (), params) for b in range(busy)]
        gates += [W.Gate("cz", (b, b + 1)) for b in range(i & 1, busy - 1, 2)]
    return gates


@functools.lru_cache(maxsize=2)
def reference(n, busy, gate, layers):
    return orc.run_circuit(W.Circuit(n, layers_of(*GATES[gate], busy, layers), x0=1))


# An operation rounds each amplitude a few times: its error is below 4 ulp of
# the norm, and errors of unitary operations add up at most linearly.
@pytest.mark.parametrize("n,busy,up", [(10, 10, 0), (11, 11, 0), (12, 12, 0), (13, 13, 0), (13, 4, 7), (18, 4, 0)])
@pytest.mark.parametrize("gate", sorted(GATES))
@pytest.mark.parametrize("prec,ulp", [(0, 2.0 ** -24), (1, 2.0 ** -53)])
def test_deep_layers(prec, ulp, n, busy, up, gate):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_09326_amd as q
    for layers in (100, 1000 if n < 18 else 300):
        gates = layers_of(*GATES[gate], busy, layers)
        sim = q.Simulator(n, prec)
        sim.init_basis(1)
        sim.run(q.Plan(n, gates, precision=prec, tile_upper=up))
        got = sim.state().astype(np.complex128)
        sim.close()
        assert np.linalg.norm(got - reference(n, busy, gate, layers)) <= 4 * len(gates) * ulp, layers
