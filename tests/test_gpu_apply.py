"""qops_apply in a row without waiting in between: the handle's program block
is rewritten in stream order and grows with the gate lists, on the default and
on a stream of its own, two handles at once."""
import numpy as np
import pytest

from oracle import oracle as orc
from workloads import circuits as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tol", [(0, 5e-5), (1, 1e-12)])
@pytest.mark.parametrize("own_stream", [False, True])
def test_calls_in_a_row(prec, tol, own_stream):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_09326_amd as q
    ns = (12, 14)
    # growing and shrinking programs; the last ones exceed the first block
    lens = (5, 60, 3, 400, 20, 1500, 2, 700)
    streams = [torch.cuda.Stream() if own_stream else None for _ in ns]
    sims = [q.Simulator(n, prec, stream=s) for n, s in zip(ns, streams)]
    parts = {n: [W.random_mixed(1000 * n + i, n, k, max_dense_k=4).gates for i, k in enumerate(lens)] for n in ns}
    for s in sims:
        s.init_basis(3)
    for i in range(len(lens)):
        for n, s in zip(ns, sims):
            s.apply(parts[n][i])
    for n, s in zip(ns, sims):
        got = s.state().astype(np.complex128)
        s.close()
        ref = orc.run_circuit(W.Circuit(n, [g for p in parts[n] for g in p], x0=3))
        assert np.max(np.abs(got - ref)) <= tol
