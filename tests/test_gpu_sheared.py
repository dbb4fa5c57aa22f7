"""Register tile passes with chains of 2x2 operations (the sheared forms):
every coefficient type (complex, real, imaginary), pivots at and around the
boundary between the plain and the exchanged form, register bits with
exchanged slots under controls, phases, general diagonals, X and LDS remaps,
and chains that end in a non-unitary 2x2.  Element by element against the
oracle with the parity bounds of the other state tests (2e-5 / 1e-12)."""
import numpy as np
import pytest

from oracle import oracle as orc
from workloads import circuits as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def q():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_09326_amd as qq
    qq.lib()
    return qq


def chain_circuit(seed, n, layers, kinds):
    """Per layer one 2x2 of a drawn kind on every qubit (angles at the pivot
    boundary and its neighbours among them), then operations that read the
    slot index: CZ, CP, RZZ, CX, a doubly controlled RY and an X."""
    rng = np.random.default_rng(seed)
    special = [0.0, np.pi / 2, np.nextafter(np.pi / 2, 4), np.nextafter(np.pi / 2, 0), np.pi, 3 * np.pi / 2]
    g = []
    for _ in range(layers):
        for b in range(n):
            kind = kinds[int(rng.integers(len(kinds)))]
            th = special[int(rng.integers(6))] if rng.random() < 0.3 else float(rng.uniform(0, 2 * np.pi))
            params = {"h": (), "sx": (), "u3": (th, *map(float, rng.uniform(0, 6.28, 2)))}.get(kind, (th,))
            g.append(W.Gate(kind, (b,), (), params))
        p = [int(v) for v in rng.permutation(n)]
        g.append(W.Gate("cz", (p[0], p[1])))
        g.append(W.Gate("cp", (p[2], p[3]), (), (0.7,)))
        g.append(W.Gate("rzz", (p[4], p[5]), (), (1.1,)))
        g.append(W.Gate("rzz", (p[5], p[6]), (), (0.3,)))
        g.append(W.Gate("cx", (p[7], p[8])))
        g.append(W.Gate("ry", (p[9],), (p[10], p[11]), (0.9,)))
        g.append(W.Gate("x", (p[12],)))
    return g


@pytest.mark.parametrize("prec,tol", [(0, 2e-5), (1, 1e-12)])
@pytest.mark.parametrize("tile_upper", [0, 4, 5, 6, 7])
@pytest.mark.parametrize("kinds", [("u3",), ("ry", "h"), ("rx", "sx"), ("u3", "ry", "rx", "h", "rz")])
def test_chains_match_oracle(q, prec, tol, tile_upper, kinds):
    n = 14
    c = W.Circuit(n, chain_circuit(len(kinds) + tile_upper, n, 5, kinds), x0=1234)
    sim = q.Simulator(n, prec)
    sim.init_basis(c.x0)
    sim.run(q.Plan(n, c.gates, precision=prec, tile_upper=tile_upper))
    got = sim.state().astype(np.complex128)
    sim.close()
    assert np.max(np.abs(got - orc.run_circuit(c))) <= tol


@pytest.mark.parametrize("prec,tol", [(0, 2e-5), (1, 1e-12)])
def test_chain_ends_in_a_singular_matrix(q, prec, tol):
    """A projector (and a scaled 2x2) after unitary 2x2s on the same bits:
    both absorb the waiting diagonal but start no chain of their own."""
    n = 13
    proj = np.array([[1.0, 0.0], [0.0, 0.0]], dtype=complex)
    big = np.array([[0.3, 1.2j], [0.1, 2.0]], dtype=complex)
    g = [W.Gate("u3", (b,), (), (0.3 + 0.2 * b, 1.0, 0.4)) for b in range(n)]
    g += [W.Gate("cz", (b, b + 1)) for b in range(n - 1)]
    g += [W.Gate("u3", (b,), (), (2.0 + 0.1 * b, 0.2, 0.9)) for b in range(n)]
    g += [W.Gate("cz", (b, (b + 3) % n)) for b in range(n)]
    g += [W.Gate("dense", (b,), (), (), proj if b in (2, 9) else big) for b in (2, 5, 9, 12)]
    g += [W.Gate("cz", (0, 12)), W.Gate("ry", (5,), (), (0.4,)), W.Gate("ry", (12,), (), (0.8,))]
    c = W.Circuit(n, g)
    sim = q.Simulator(n, prec)
    sim.init_basis(0)
    sim.apply(c.gates)
    got = sim.state().astype(np.complex128)
    sim.close()
    assert np.max(np.abs(got - orc.run_circuit(c))) <= tol


@pytest.mark.parametrize("prec,tol", [(0, 2e-5), (1, 1e-12)])
@pytest.mark.parametrize("n,tile_upper", [(10, 0), (11, 0), (12, 0), (13, 0), (13, 4), (13, 5), (13, 6), (13, 7)])
def test_every_register_condition(q, prec, tol, n, tile_upper):
    """CZ, CP, CX and RZZ on every pair of qubits, triple phases and a
    four-bit diagonal between layers of 2x2s (so that register bits are met
    with slots in order and exchanged): the bodies compiled per register bit,
    pair and required value, the general ones, and 10..12-qubit states that
    are one register tile."""
    rng = np.random.default_rng(n + 100 * tile_upper)
    g = []
    pairs = [(int(a), int(b)) for a in range(n) for b in range(n) if a != b]
    rng.shuffle(pairs)
    for i, (a, b) in enumerate(pairs):
        if i % 12 == 0:
            g += [W.Gate("u3", (b2,), (), tuple(map(float, rng.uniform(0, 6.28, 3)))) for b2 in range(n)]
        g.append(W.Gate(("cz", "cx", "cp", "rzz")[i % 4], (a, b), (), (float(rng.uniform(0, 6.28)),) if i % 4 > 1 else ()))
        if i % 9 == 4:
            c = int(rng.choice([v for v in range(n) if v not in (a, b)]))
            g.append(W.Gate("z" if i % 2 else "p", (a,), (b, c), () if i % 2 else (0.8,)))
            g.append(W.Gate("x", (c,), (a, b)))
        if i % 17 == 3:
            c, d = (int(v) for v in rng.choice([v for v in range(n) if v not in (a, b)], 2, replace=False))
            g += [W.Gate("rzz", (a, c), (), (0.3,)), W.Gate("rzz", (c, d), (), (0.5,)), W.Gate("rzz", (d, b), (), (0.7,))]
    circ = W.Circuit(n, g, x0=5)
    sim = q.Simulator(n, prec)
    sim.init_basis(5)
    sim.run(q.Plan(n, g, precision=prec, tile_upper=tile_upper))
    got = sim.state().astype(np.complex128)
    sim.close()
    assert np.max(np.abs(got - orc.run_circuit(circ))) <= tol


@pytest.mark.parametrize("prec,tol", [(0, 2e-5), (1, 1e-12)])
@pytest.mark.parametrize("n,tile_upper", [(10, 0), (13, 0), (14, 4), (14, 5), (14, 6), (14, 7)])
@pytest.mark.parametrize("kind", ["u3", "ry", "rx"])
def test_row_swaps(q, prec, tol, n, tile_upper, kind):
    """2x2s on lane bits 2..5 alone and on register bits between them: each
    order and exchange of the row-swapped form (angles on both sides of the
    pivot boundary), the slots it leaves exchanged read by controls, phases,
    X, RZZ and remaps."""
    rng = np.random.default_rng(10 * n + tile_upper)
    g = [W.Gate("h", (b,)) for b in range(n)]
    for i in range(30):
        for b in (2, 3, 4, 5):
            th = float((0.4, 2.7, np.pi, -2.0, 0.0, 4.4)[int(rng.integers(6))])
            g.append(W.Gate(kind, (b,), (), (th, *map(float, rng.uniform(0, 6.28, 2))) if kind == "u3" else (th,)))
        b, c = (int(v) for v in rng.choice(np.arange(4, n), 2, replace=False))
        k = ("cz", "cx", "cp", "rzz", "x")[i % 5]
        g.append(W.Gate(k, (b,) if k == "x" else (b, c), (), (0.9,) if k in ("cp", "rzz") else ()))
        if i % 4 == 0:
            g.append(W.Gate("u3", (int(rng.integers(6, n)),), (), (float(rng.uniform(0, 6.28)), 0.3, 1.2)))
    circ = W.Circuit(n, g, x0=3)
    sim = q.Simulator(n, prec)
    sim.init_basis(circ.x0)
    sim.run(q.Plan(n, circ.gates, precision=prec, tile_upper=tile_upper))
    got = sim.state().astype(np.complex128)
    sim.close()
    assert np.max(np.abs(got - orc.run_circuit(circ))) <= tol


@pytest.mark.parametrize("prec,tol", [(0, 2e-5), (1, 1e-12)])
@pytest.mark.parametrize("n,tile_upper", [(10, 0), (12, 0), (14, 4), (14, 5), (14, 6), (14, 7)])
def test_diagonal_tables(q, prec, tol, n, tile_upper):
    """Tables of 1 to 6 bits with bits in lanes, registers (exchanged or not),
    waves and outside the tile, in ascending and descending order: the ones in
    a record and the ones in the coefficient array.  Every entry of a table is
    different, so a swapped bit shows."""
    rng = np.random.default_rng(7 * n + tile_upper)
    g = [W.Gate("u3", (b,), (), (1.0 + 0.1 * b, 0.2, 0.5)) for b in range(n)]
    for i in range(60):
        k = 1 + i % 6
        w = [int(v) for v in rng.choice(n, k, replace=False)]
        if k == 1:
            g.append(W.Gate("p", (w[0],), (), (float(rng.uniform(0, 6.28)),)))
        for j in range(k - 1):
            g.append(W.Gate("rzz", (w[j], w[j + 1]), (), (float(rng.uniform(0, 6.28)),)))
            g.append(W.Gate("rz", (w[j],), (), (float(rng.uniform(0, 6.28)),)))
        for b in (int(v) for v in rng.choice(n, 3, replace=False)):
            g.append(W.Gate(("u3", "rx", "ry")[i % 3], (b,), (),
                            tuple(map(float, rng.uniform(0, 6.28, 3 if i % 3 == 0 else 1)))))
    circ = W.Circuit(n, g, x0=9)
    sim = q.Simulator(n, prec)
    sim.init_basis(circ.x0)
    sim.run(q.Plan(n, circ.gates, precision=prec, tile_upper=tile_upper))
    got = sim.state().astype(np.complex128)
    sim.close()
    assert np.max(np.abs(got - orc.run_circuit(circ))) <= tol


@pytest.mark.parametrize("prec,tol", [(0, 2e-5), (1, 1e-12)])
@pytest.mark.parametrize("n,tile_upper", [(10, 0), (14, 4), (14, 5), (14, 6), (14, 7)])
def test_x_on_lanes(q, prec, tol, n, tile_upper):
    """X on each lane bit, alone and under controls in lanes, registers, waves
    and outside the tile (one and two of them)."""
    g = [W.Gate("u3", (b,), (), (1.0 + 0.1 * b, 0.2, 0.5)) for b in range(n)]
    for b in range(6):
        g += [W.Gate("cz", (b, (b + 1) % 6)), W.Gate("x", (b,)), W.Gate("cp", (b, n - 1), (), (0.4,))]
        for c in range(n):
            if c == b:
                continue
            g.append(W.Gate("cx", (c, b)))
            g.append(W.Gate("cp", (b, (b + 3) % 6), (), (0.2 + 0.1 * c,)))
            if c % 3 == 0 and (c + 5) % n != b:
                g.append(W.Gate("x", (b,), (c, (c + 5) % n)))
                g.append(W.Gate("ry", (b,), (), (0.3,)))
    circ = W.Circuit(n, g, x0=6)
    sim = q.Simulator(n, prec)
    sim.init_basis(circ.x0)
    sim.run(q.Plan(n, circ.gates, precision=prec, tile_upper=tile_upper))
    got = sim.state().astype(np.complex128)
    sim.close()
    assert np.max(np.abs(got - orc.run_circuit(circ))) <= tol


@pytest.mark.parametrize("n,tile_upper", [(21, 7), (22, 6), (23, 6), (24, 7)])
def test_default_width_against_another(q, n, tile_upper):
    """The default register tile on both sides of the sizes where its width
    changes, against an explicit other width: the same state to rounding
    (both within 2e-5 of the oracle by the other tests, so within 4e-5 here)."""
    rng = np.random.default_rng(n)
    g = []
    for _ in range(4):
        g += [W.Gate("u3", (b,), (), tuple(map(float, rng.uniform(0, 6.28, 3)))) for b in range(n)]
        p = [int(v) for v in rng.permutation(n)]
        g += [W.Gate(("cz", "cx", "rzz")[i % 3], (p[2 * i], p[2 * i + 1]), (), (0.7,) if i % 3 == 2 else ())
              for i in range(n // 2)]
    out = []
    for up in (0, tile_upper):
        sim = q.Simulator(n, 0)
        sim.init_basis(7)
        sim.run(q.Plan(n, g, precision=0, tile_upper=up))
        out.append(sim.state())
        sim.close()
    assert np.max(np.abs(out[0] - out[1])) <= 4e-5


@pytest.mark.parametrize("n", [12, 16, 20])
@pytest.mark.parametrize("angle", [0.3, 0.9, 1.7, 2.6])
def test_one_angle_on_every_qubit_keeps_the_norm(q, n, angle):
    """The rounding of a 2x2's coefficients is the same for every qubit under
    one angle, so it must not add up in the norm: what is left is one rounded
    factor a pass and a few units of the last place (2^-24 each)."""
    g = [W.Gate("h", (b,)) for b in range(n)]
    for layer in range(4):
        g += [W.Gate("rzz", (b, (b + 1) % n), (), (0.37 + 0.1 * b + layer,)) for b in range(n)]
        g += [W.Gate("rx" if layer % 2 else "ry", (b,), (), (angle,)) for b in range(n)]
    sim = q.Simulator(n, 0)
    sim.init_basis(0)
    p = q.Plan(n, g, precision=0)
    sim.run(p)
    norm = np.linalg.norm(sim.state().astype(np.complex128))
    sim.close()
    assert abs(norm - 1) <= (p.stats()["n_passes"] + 6) * 2.0 ** -24
