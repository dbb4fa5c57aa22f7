"""Batched circuits that run as one register tile (10..13 qubits, a graph
branch per kernel) beside LDS circuits (fewer qubits, or a dense block) and
tile-pass circuits: <Z> against the oracle, replays, and new parameters."""
import numpy as np
import pytest

from oracle import oracle as orc
from workloads import circuits as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tol,top", [(0, 2e-5, 13), (1, 1e-11, 12)])
def test_whole_state_tiles(prec, tol, top):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_09326_amd as q
    rng = np.random.default_rng(prec)
    circs = []
    for n in (*range(9, top + 1), 15, 16):
        circs += W.param_sweep_batch(seed=n, count=2, nmin=n, nmax=n, dmin=3, dmax=9)
    # a dense block keeps a circuit of that width in the LDS kernel
    g = list(circs[4].gates) + [W.Gate("dense", (1, 3), (), (), W.haar_unitary(W.rng_for(3), 4))]
    circs.append(W.Circuit(circs[4].n, g))
    b = q.Batch([(c.n, c.gates) for c in circs], precision=prec)
    assert b.info()["tile_circuits"] == 4
    for _ in range(2):
        b.launch()
        first = b.results()
        for c, z in zip(circs, first):
            assert np.max(np.abs(z - orc.expect_z(orc.run_circuit(c)))) <= tol
        torch.cuda.synchronize()
    new = [W.Circuit(c.n, [W.Gate(x.kind, x.qubits, x.controls, tuple(rng.uniform(0, 6.28, len(x.params))), x.matrix)
                           for x in c.gates]) for c in circs]
    b.update([c.gates for c in new])
    b.launch()
    for c, z in zip(new, b.results()):
        assert np.max(np.abs(z - orc.expect_z(orc.run_circuit(c)))) <= tol
    b.close()
