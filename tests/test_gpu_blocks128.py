"""complex128 blocks of 2 to 6 qubits in the LDS tile pass: the full tile of
2^12 amplitudes runs eight waves and reads every coefficient from LDS.  Each
block size with and without a control and beside diagonals, on the full tile
and on smaller ones (four waves), one work-group walking every tile and the
default grid.  Tolerance of the whole suite: max-abs <= 1e-12.  On the CPU:
every plan of mixed blocks and diagonals stages what it has to."""
import numpy as np
import pytest

from oracle import oracle as orc
from workloads import circuits as W

TOL = 1e-12


def haar(rng, k):
    q, r = np.linalg.qr(rng.standard_normal((2 ** k, 2 ** k)) + 1j * rng.standard_normal((2 ** k, 2 ** k)))
    d = np.diagonal(r)
    return q * (d / np.abs(d))


def gates(n, k, seed):
    rng = np.random.default_rng(seed)
    out = []
    for i in range(5):
        w = [int(v) for v in rng.choice(n, k + 1, replace=False)]
        out.append(W.Gate("dense", tuple(w[:k]), (w[k],) if i % 2 else (), (), haar(rng, k)))
        if i % 2:
            d = [int(v) for v in rng.choice(n, 3, replace=False)]
            out.append(W.Gate("rzz", (d[0], d[1]), (), (0.7,)))
            out.append(W.Gate("cp", (d[1], d[2]), (), (1.1,)))
            out.append(W.Gate("ry", (d[2],), (), (0.3,)))
    return out


@pytest.mark.parametrize("k", [2, 3, 4, 5, 6])
@pytest.mark.parametrize("n", [13, 18, 23])
def test_every_plan_is_staged(k, n):
    import paper_2410_09326_amd as q
    for seed in range(8):
        g = gates(n, k, 10 * k + seed) + gates(n, 2 + seed % 5, seed)
        for opts in ({}, {"merge_blocks": -1}, {"tile_upper": 5}, {"use_mfma": 0}):
            p = q.Plan(n, q.GateArray(g), precision=q.C128, **opts)
            assert p.stats()["n_passes"] > 0


@pytest.mark.gpu
@pytest.mark.parametrize("k", [2, 3, 4, 5, 6])
@pytest.mark.parametrize("n,limit", [(13, 1), (15, 3), (15, 0)])
@pytest.mark.parametrize("opts", [{}, {"tile_upper": 5}, {"merge_blocks": -1}])
def test_blocks(k, n, limit, opts):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_09326_amd as q
    g = gates(n, k, 100 * n + k)
    x0 = 5 % (1 << n)
    ref = orc.run(n, g, x0=x0)
    sim = q.Simulator(n, q.C128)
    sim.set_launch_limit(limit)
    sim.init_basis(x0)
    sim.apply(q.GateArray(g), **opts)
    got = sim.state()
    sim.close()
    assert np.max(np.abs(got - ref)) <= TOL
