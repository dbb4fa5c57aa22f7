"""Batched circuits that one work-group runs start to finish, up to 128 layers
deep and beside each other: <Z> against the oracle, replays, new parameters;
and every such circuit of the 512-circuit parameter sweep."""
import numpy as np
import pytest

from oracle import oracle as orc
from workloads import circuits as W

pytestmark = pytest.mark.gpu


def sweep(n, depth, seed):
    return W.param_sweep_batch(seed=seed, count=1, nmin=n, nmax=n, dmin=depth, dmax=depth)[0]


# four ulp of the state's norm per operation, added up, and |d<Z>| <= 2 |dpsi|
@pytest.mark.parametrize("prec,ulp", [(0, 2.0 ** -24), (1, 2.0 ** -53)])
@pytest.mark.parametrize("shape", [((13, 24), (13, 64), (13, 128)), ((10, 250), (11, 170), (12, 130), (13, 21), (13, 40)),
                                   ((9, 40), (12, 60), (13, 33), (14, 12), (16, 9), (10, 8))])
def test_deep_batch(shape, prec, ulp):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_09326_amd as q
    rng = np.random.default_rng(len(shape))
    circs = [sweep(n, d, 10 * i + d) for i, (n, d) in enumerate(shape)]
    b = q.Batch([(c.n, c.gates) for c in circs], precision=prec)
    for _ in range(2):
        for _ in range(3):
            b.launch()
            for c, z in zip(circs, b.results()):
                assert np.max(np.abs(z - orc.expect_z(orc.run_circuit(c)))) <= 8 * len(c.gates) * ulp, c.n
            torch.cuda.synchronize()
        circs = [W.Circuit(c.n, [W.Gate(x.kind, x.qubits, x.controls, tuple(rng.uniform(0, 6.28, len(x.params))))
                                 for x in c.gates]) for c in circs]
        b.update([c.gates for c in circs])
    b.close()


def test_sweep_whole_state_circuits():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_09326_amd as q
    circs = W.param_sweep_batch()
    b = q.Batch([(c.n, c.gates) for c in circs], precision=q.C64)
    b.launch()
    res = b.results()
    b.close()
    whole = [i for i, c in enumerate(circs) if c.n <= 13]
    assert len(whole) > 100
    for i in whole:
        c = circs[i]
        assert np.max(np.abs(res[i] - orc.expect_z(orc.run_circuit(c)))) <= 8 * len(c.gates) * 2.0 ** -24, (i, c.n)
