"""Readout reductions at the edges of their geometry (states smaller than a
row, fewer than eight rows, one and several chunks, every split of marginal
bits into row, walked, sliced and numbering bits), both precisions, after a
layout change, against FP64 sums over the amplitudes the device holds."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def q():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_09326_amd as qq
    qq.lib()
    return qq


def held_state(q, n, prec, offset=0):
    """A simulator with a random state and a shuffled layout, and the
    probabilities in logical order."""
    import torch
    rng = np.random.default_rng(100 * n + prec + offset)
    psi = rng.normal(size=2 ** n) + 1j * rng.normal(size=2 ** n)
    psi = (psi / np.linalg.norm(psi)).astype(np.complex64 if prec == 0 else np.complex128)
    per = 2 if prec == 0 else 4
    pad = torch.zeros(per * (2 ** n + offset), dtype=torch.float32, device="cuda:0")
    sim = q.Simulator(n, prec, buffer=pad[per * offset:])
    sim.init_amplitudes(psi)
    p = np.abs(psi.astype(np.complex128)) ** 2
    for _ in range(n // 2):
        a, b = (int(v) for v in rng.choice(n, 2, replace=False))
        sim.swap(a, b)
        x = np.arange(2 ** n)
        ba, bb = (x >> a) & 1, (x >> b) & 1
        p = p[(x & ~((1 << a) | (1 << b))) | (bb << a) | (ba << b)]
    return sim, p, rng


# the sums have 2^n terms of mean 2^-n: with any fixed order of pairwise or
# per-thread chains (at most 2^13 terms) the error stays below 2^13 * 2^-53
TOL = 2.0 ** -40


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n", [1, 2, 5, 8, 9, 10, 11, 12, 13, 16, 17, 21])
def test_marginals(q, prec, n):
    sim, p, rng = held_state(q, n, prec)
    x = np.arange(2 ** n)
    for m in sorted({1, 2, min(n, 5), max(1, n // 2), max(1, n - 9), max(1, n - 1), n}):
        if m > n:
            continue
        qs = [int(v) for v in rng.choice(n, m, replace=False)]
        y = np.zeros(2 ** n, dtype=np.int64)
        for j, b in enumerate(qs):
            y |= ((x >> b) & 1) << j
        ref = np.bincount(y, weights=p, minlength=2 ** m)
        got = sim.probabilities(qs)
        assert np.max(np.abs(got - ref)) <= TOL, (n, qs)
        assert np.array_equal(got, sim.probabilities(qs))
    sim.close()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,offset", [(1, 0), (2, 0), (6, 0), (8, 1), (9, 0), (10, 0), (11, 1), (12, 0), (15, 0), (16, 0),
                                      (17, 1), (20, 0)])
def test_z_norm_and_correlators(q, prec, n, offset):
    sim, p, rng = held_state(q, n, prec, offset)
    x = np.arange(2 ** n)
    sgn = [1.0 - 2.0 * ((x >> b) & 1) for b in range(n)]
    assert np.max(np.abs(sim.expect_z() - np.array([np.dot(s, p) for s in sgn]))) <= TOL
    assert abs(sim.norm() - p.sum()) <= TOL
    # every pair and some of a qubit with itself: several launches of 64
    pairs = [(a, b) for a in range(n) for b in range(a + 1, n)] + [(n - 1, n - 1), (0, 0)]
    rng.shuffle(pairs)
    ref = np.array([np.dot(sgn[a] * sgn[b], p) for a, b in pairs])
    got = sim.expect_zz(pairs)
    assert np.max(np.abs(got - ref)) <= TOL
    assert np.array_equal(got, sim.expect_zz(pairs))
    sim.close()
