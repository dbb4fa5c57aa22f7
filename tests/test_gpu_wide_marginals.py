"""Marginals over so many bits that their work-groups need a second dimension
of the dispatch (2^20 in the first), up to 2^32 work-items and more: products of single-qubit distributions, so the oracle is a product."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,prec,qubits", [
    (30, 0, list(range(9, 30))),                     # 2^21 work-groups
    (30, 0, [3, 8] + list(range(10, 30)) + [0]),     # 2^20, row bits among the outputs
    (31, 0, list(range(30, 8, -1))),                 # 2^22, reversed
    (29, 1, [1] + list(range(8, 29))),               # complex128, no free bit above a row
    (33, 0, list(range(9, 33))),                     # 2^24: 2^32 work-items
])
def test_wide_marginals(n, prec, qubits):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_09326_amd as q
    theta = np.linspace(1.2, 1.9, n)                 # amplitudes positive: no cancellation
    sim = q.Simulator(n, prec)
    sim.init_basis(0)
    sim.run(q.Plan(n, [("ry", (b,), (float(theta[b]),)) for b in range(n)], precision=prec))
    got = sim.probabilities(qubits)
    sim.close()
    del sim
    torch.cuda.empty_cache()
    ref = np.ones(1)
    for b in qubits:
        ref = np.concatenate([ref * np.cos(theta[b] / 2) ** 2, ref * np.sin(theta[b] / 2) ** 2])
    # n operations of four ulp each, squared
    ulp = 2.0 ** -24 if prec == 0 else 2.0 ** -53
    assert np.max(np.abs(got / ref - 1)) <= 8 * (n + 1) * ulp
