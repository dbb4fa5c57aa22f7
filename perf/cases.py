"""The work that users of the simulator time: whole circuits through a kept
plan or in one call, repeated parameter runs, a batch of small circuits, and
the readouts of a large state.

A case names one call pattern with its sizes; `prepare` builds what a program
holds before the call (state buffer, plan, gate arrays), `run` is one pass
through the public entry points, `exact` the same result from plain torch in
64 bits.  Sizes follow the repository's benchmark and tests: the 12-qubit
layered circuit, the 28-qubit QFT with layers, the 30-qubit Haar blocks, the
cost-model corpus (20..30 qubits), the 28-qubit Max-Cut QAOA, the parameter
sweep (10..22 qubits) and their odd and ragged neighbours.

Complex64 circuits return the state itself.  <Z> and <ZZ> values read from a
complex64 circuit are returned as float32, the precision they carry; the
readout cases start from a given state, so theirs are float64.
"""
import math

import numpy as np
import torch

import paper_2410_09326_amd as q

DEVICE = "cuda:0"


def listed():
    return [
        # smallest calls: a 12-qubit layered circuit on a kept plan (the
        # oracle-checked reference workload, complex128)
        {"name": "layered12_c128", "op": "circuit", "kind": "layered", "n": 12, "size": 20, "prec": "c128", "how": "plan"},
        # a small circuit in one call, planned each time (interactive use)
        {"name": "apply_clifft15_c64", "op": "circuit", "kind": "clifft", "n": 15, "size": 400, "prec": "c64", "how": "apply"},
        # an ordinary mixed circuit whose state stays in cache
        {"name": "mix20_c64", "op": "circuit", "kind": "mix", "n": 20, "size": 40, "prec": "c64", "how": "plan"},
        # gate-level circuits on large states
        {"name": "qft28_layers40_c64", "op": "circuit", "kind": "qft", "n": 28, "size": 40, "prec": "c64", "how": "plan"},
        {"name": "mix25_c128", "op": "circuit", "kind": "mix", "n": 25, "size": 40, "prec": "c128", "how": "plan"},
        # dense blocks on matrix cores: the benchmark circuit, and complex128
        {"name": "haar30_c64", "op": "circuit", "kind": "haar", "n": 30, "size": 200, "prec": "c64", "how": "plan"},
        {"name": "haar23_c128", "op": "circuit", "kind": "haar", "n": 23, "size": 60, "prec": "c128", "how": "plan"},
        # repeated runs: new angles on one plan, the state and every edge's <ZZ>
        {"name": "qaoa28_c64", "op": "qaoa", "n": 28, "size": 3, "prec": "c64"},
        # a parameter sweep of uneven circuits in one graph launch
        {"name": "batch96_c64", "op": "batch", "n": 10, "nmax": 20, "size": 96, "prec": "c64"},
        # readouts: every <Z> of the largest benchmark state, the distribution
        # of a few qubits, and a wide marginal of an odd-sized complex128 state
        {"name": "expect_z30_c64", "op": "expect_z", "n": 30, "prec": "c64"},
        {"name": "probs8of28_c64", "op": "probs", "n": 28, "size": 8, "prec": "c64"},
        {"name": "probs15of25_c128", "op": "probs", "n": 25, "size": 15, "prec": "c128"},
    ]


def draw(rng):
    prec = rng.choice(["c64", "c64", "c128"])
    less = 1 if prec == "c128" else 0

    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["circuit"] * 6 + ["qaoa", "batch", "expect_z", "probs", "zz"])
    if op == "circuit":
        kind = rng.choice(["layered", "clifft", "mix", "qft", "haar"])
        how = rng.choice(["plan", "plan", "apply"])
        if kind == "layered":
            return {"op": op, "kind": kind, "n": rng.randint(4, 18), "size": log_int(3, 40), "prec": prec, "how": how}
        if kind == "clifft":
            return {"op": op, "kind": kind, "n": rng.randint(5, 24), "size": log_int(40, 800), "prec": prec, "how": how}
        if kind == "mix":
            return {"op": op, "kind": kind, "n": rng.randint(18, 27) - less, "size": log_int(10, 80), "prec": prec, "how": how}
        if kind == "qft":
            return {"op": op, "kind": kind, "n": rng.randint(13, 27) - less, "size": log_int(1, 40), "prec": prec, "how": how}
        return {"op": op, "kind": kind, "n": rng.randint(13, 27) - less, "size": log_int(10, 120), "prec": prec, "how": how}
    if op == "qaoa":
        return {"op": op, "n": 2 * rng.randint(5, 13), "size": rng.randint(1, 5), "prec": prec}
    if op == "batch":
        n = rng.randint(5, 12)
        return {"op": op, "n": n, "nmax": n + rng.randint(1, 7), "size": log_int(6, 64), "prec": prec}
    n = rng.randint(9, 29) - less
    if op == "probs":
        return {"op": op, "n": n, "size": rng.randint(1, min(n, 20)), "prec": prec}
    if op == "zz":
        return {"op": op, "n": n, "size": log_int(1, 80), "prec": prec}
    return {"op": op, "n": n, "prec": prec}


# --------------------------------------------------------------------------
# Circuits as (kind, qubits, params, controls, matrix) tuples
# --------------------------------------------------------------------------

def _haar(rng, d):
    z = rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d))
    u, r = np.linalg.qr(z)
    g = np.diagonal(r)
    return u * (g / np.abs(g))[None, :]


def _angles(rng, k):
    return tuple(float(v) for v in rng.uniform(0.0, 2.0 * np.pi, k))


def _pairs(rng, n):
    p = [int(v) for v in rng.permutation(n)]
    return [(p[2 * i], p[2 * i + 1]) for i in range(n // 2)], p[2 * (n // 2):]


def _layered(rng, n, depth):
    """U3 on every qubit and CNOTs on a random pairing; a SWAP in a tenth of
    the layers."""
    g = []
    swaps = set(int(v) for v in rng.choice(depth, size=int(round(0.1 * depth)), replace=False))
    for layer in range(depth):
        g += [("u3", (b,), _angles(rng, 3)) for b in range(n)]
        g += [("cx", pr) for pr in _pairs(rng, n)[0]]
        if layer in swaps:
            g.append(("swap", tuple(int(v) for v in rng.choice(n, size=2, replace=False))))
    return g


def _clifft(rng, n, count):
    """Clifford+T stream with 30 % T gates."""
    g = []
    for _ in range(count):
        if rng.random() < 0.3:
            g.append(("t" if rng.random() < 0.5 else "tdg", (int(rng.integers(n)),)))
            continue
        kind = ("h", "s", "x", "z", "cx", "cx", "cz")[int(rng.integers(7))]
        k = 2 if kind in ("cx", "cz") else 1
        g.append((kind, tuple(int(v) for v in rng.choice(n, size=k, replace=False))))
    return g


def _mix(rng, n, depth):
    """Per layer one of U3 x U3, CZ, SWAP, RZZ on every pair of a random
    pairing."""
    g = []
    for _ in range(depth):
        pairs, rest = _pairs(rng, n)
        for a, b in pairs:
            c = int(rng.integers(4))
            if c == 0:
                g += [("u3", (a,), _angles(rng, 3)), ("u3", (b,), _angles(rng, 3))]
            elif c == 1:
                g.append(("cz", (a, b)))
            elif c == 2:
                g.append(("swap", (a, b)))
            else:
                g.append(("rzz", (a, b), _angles(rng, 1)))
        g += [("u3", (b,), _angles(rng, 3)) for b in rest]
    return g


def _qft(rng, n, layers):
    """QFT, then layers of U3 on every qubit and CZ on a random pairing."""
    g = []
    for j in range(n - 1, -1, -1):
        g.append(("h", (j,)))
        g += [("cp", (m, j), (math.pi / 2 ** (j - m),)) for m in range(j - 1, -1, -1)]
    g += [("swap", (i, n - 1 - i)) for i in range(n // 2)]
    for _ in range(layers):
        g += [("u3", (b,), _angles(rng, 3)) for b in range(n)]
        g += [("cz", pr) for pr in _pairs(rng, n)[0]]
    return g


def _haar_blocks(rng, n, blocks):
    """Haar-random dense blocks of 2..6 qubits on random qubits."""
    g = []
    for _ in range(blocks):
        k = int(rng.integers(2, 7))
        qs = tuple(int(v) for v in rng.choice(n, size=k, replace=False))
        g.append(("dense", qs, (), (), _haar(rng, 2 ** k)))
    return g


def _edges(rng, n):
    """A random 3-regular simple graph (pairing model) and edge weights."""
    while True:
        s = np.repeat(np.arange(n), 3)
        rng.shuffle(s)
        e = {(int(min(a, b)), int(max(a, b))) for a, b in s.reshape(-1, 2)}
        if len(e) == 3 * n // 2 and all(a != b for a, b in e):
            return sorted(e), rng.uniform(0.5, 1.5, len(e))


def _qaoa(rng, n, edges, w, p):
    g = [("h", (b,)) for b in range(n)]
    for _ in range(p):
        gm, bt = float(rng.uniform(0.1, 1.2)), float(rng.uniform(0.1, 0.8))
        g += [("rzz", e, (-gm * float(x),)) for e, x in zip(edges, w)]
        g += [("rx", (b,), (2.0 * bt,)) for b in range(n)]
    return g


def _sweep(rng, n, depth):
    """RY and RZ on every qubit, then a CZ ladder."""
    g = []
    for _ in range(depth):
        a = rng.uniform(0.0, 2.0 * np.pi, (n, 2))
        for b in range(n):
            g += [("ry", (b,), (float(a[b, 0]),)), ("rz", (b,), (float(a[b, 1]),))]
        g += [("cz", (b, b + 1)) for b in range(n - 1)]
    return g


_MAKE = {"layered": _layered, "clifft": _clifft, "mix": _mix, "qft": _qft, "haar": _haar_blocks}


def _circuit(case, seed):
    rng = np.random.default_rng([seed, case["n"], case["size"]])
    x0 = int(rng.integers(2 ** case["n"]))
    return x0, _MAKE[case["kind"]](rng, case["n"], case["size"])


def _qaoa_inputs(case, seed):
    rng = np.random.default_rng([seed, case["n"], case["size"]])
    edges, w = _edges(rng, case["n"])
    first = _qaoa(rng, case["n"], edges, w, case["size"])
    return edges, first, _qaoa(rng, case["n"], edges, w, case["size"])


def _batch_inputs(case, seed):
    """Widths and depths belong to the case, the angles to the seed."""
    shape = np.random.default_rng([case["n"], case["nmax"], case["size"]])
    rng = np.random.default_rng([seed, case["n"], case["size"]])
    out = []
    for _ in range(case["size"]):
        n = int(shape.integers(case["n"], case["nmax"] + 1))
        out.append((n, _sweep(rng, n, int(shape.integers(8, 33)))))
    return out


def _random_state(case, seed):
    """A normalised random state in physical order (interleaved re, im), the
    swaps that set its layout, and the qubits or pairs a readout asks for."""
    n = case["n"]
    rng = np.random.default_rng([seed, n, case.get("size", 0)])
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    dt = torch.float32 if case["prec"] == "c64" else torch.float64
    buf = torch.empty(2 ** (n + 1), dtype=dt, device=DEVICE)
    buf.normal_(generator=gen)
    buf.mul_(2.0 ** (-0.5 * (n + 1)))
    swaps = [tuple(int(v) for v in rng.choice(n, size=2, replace=False)) for _ in range(n // 2)]
    asked = None
    if case["op"] == "probs":
        asked = [int(v) for v in rng.choice(n, size=case["size"], replace=False)]
    elif case["op"] == "zz":
        asked = [tuple(int(v) for v in rng.choice(n, size=2, replace=False)) for _ in range(case["size"])]
    return buf, swaps, asked


# --------------------------------------------------------------------------
# One pass through the public entry points
# --------------------------------------------------------------------------

def _prec(case):
    return q.C64 if case["prec"] == "c64" else q.C128


def _amplitudes(sim):
    return sim.buffer if sim.precision == q.C64 else sim.buffer.view(torch.float64)


def prepare(case, seed):
    op, n, prec = case["op"], case["n"], _prec(case)
    if op == "circuit":
        x0, gates = _circuit(case, seed)
        s = {"sim": q.Simulator(n, prec, device=DEVICE), "x0": x0}
        if case["how"] == "plan":
            s["plan"] = q.Plan(n, gates, precision=prec)
        else:
            s["gates"] = q.GateArray(gates)
        return dict(s, op=case["how"])
    if op == "qaoa":
        edges, first, gates = _qaoa_inputs(case, seed)
        return {"op": op, "sim": q.Simulator(n, prec, device=DEVICE), "plan": q.Plan(n, first, precision=prec),
                "gates": q.GateArray(gates), "edges": edges}
    if op == "batch":
        return {"op": op, "batch": q.Batch(_batch_inputs(case, seed), precision=prec),
                "single": case["prec"] == "c64"}
    buf, swaps, asked = _random_state(case, seed)
    sim = q.Simulator(n, prec, device=DEVICE, buffer=buf)
    for a, b in swaps:
        sim.swap(a, b)
    return {"op": op, "sim": sim, "asked": asked}


def run(state):
    op = state["op"]
    if op == "batch":
        state["batch"].launch()
        z = np.concatenate(state["batch"].results())
        return z.astype(np.float32) if state["single"] else z
    sim = state["sim"]
    if op == "plan":
        sim.init_basis(state["x0"])
        sim.run(state["plan"])
        return _amplitudes(sim)
    if op == "apply":
        sim.init_basis(state["x0"])
        sim.apply(state["gates"])
        return _amplitudes(sim)
    if op == "qaoa":
        state["plan"].update(state["gates"])
        sim.init_basis(0)
        sim.run(state["plan"])
        zz = sim.expect_zz(state["edges"])
        return {"state": _amplitudes(sim), "zz": zz.astype(np.float32) if sim.precision == q.C64 else zz}
    if op == "expect_z":
        return sim.expect_z()
    if op == "zz":
        return sim.expect_zz(state["asked"])
    return sim.probabilities(state["asked"])


# --------------------------------------------------------------------------
# What a pass cannot do without
# --------------------------------------------------------------------------

_DIAGONAL = ("z", "s", "sdg", "t", "tdg", "rz", "p", "cz", "cp", "rzz")


def _gate_flops(gates, n):
    total = 0.0
    for g in gates:
        kind, k = g[0], len(g[1])
        if kind in ("swap", "x", "cx"):
            continue
        if kind in ("rz", "rzz"):
            total += 6.0 * 2 ** n
        elif kind in _DIAGONAL:
            total += 6.0 * 2 ** (n - k)
        else:
            total += (8.0 * 2 ** k - 2.0) * 2 ** n
    return total


def work(case):
    n, op = case["n"], case["op"]
    amp = 8 if case["prec"] == "c64" else 16
    if op == "circuit":
        return {"bytes": amp * 2.0 ** n, "flops": _gate_flops(_circuit(case, 1)[1], n)}
    if op == "qaoa":
        edges, _, gates = _qaoa_inputs(case, 1)
        return {"bytes": amp * 2.0 ** n, "flops": _gate_flops(gates, n) + (3.0 + len(edges)) * 2 ** n}
    if op == "batch":
        circs = _batch_inputs(case, 1)
        return {"bytes": 8.0 * sum(m for m, _ in circs),
                "flops": sum(_gate_flops(g, m) + (3.0 + m) * 2.0 ** m for m, g in circs)}
    out = {"expect_z": n, "zz": case.get("size", 0), "probs": 2 ** case.get("size", 0)}[op]
    per = {"expect_z": 3.0 + n, "zz": 3.0 + case.get("size", 0), "probs": 4.0}[op]
    return {"bytes": amp * 2.0 ** n + 8.0 * out, "flops": per * 2 ** n}


# --------------------------------------------------------------------------
# The same results in 64 bits from plain torch
# --------------------------------------------------------------------------

def _matrix(g):
    kind, t = g[0], (g[2] if len(g) > 2 else ())
    e = lambda a: complex(math.cos(a), math.sin(a))  # noqa: E731
    r = math.sqrt(0.5)
    if kind == "dense":
        return np.asarray(g[4], dtype=np.complex128)
    if kind == "u3":
        c, s = math.cos(t[0] / 2), math.sin(t[0] / 2)
        m = [[c, -e(t[2]) * s], [e(t[1]) * s, e(t[1] + t[2]) * c]]
    elif kind in ("rx", "ry"):
        c, s = math.cos(t[0] / 2), math.sin(t[0] / 2)
        m = [[c, -1j * s], [-1j * s, c]] if kind == "rx" else [[c, -s], [s, c]]
    else:
        m = {"h": [[r, r], [r, -r]], "x": [[0, 1], [1, 0]], "z": [[1, 0], [0, -1]], "s": [[1, 0], [0, 1j]],
             "t": [[1, 0], [0, e(math.pi / 4)]], "tdg": [[1, 0], [0, e(-math.pi / 4)]]}.get(kind)
        if kind == "rz":
            m = [[e(-t[0] / 2), 0], [0, e(t[0] / 2)]]
    return np.array(m, dtype=np.complex128)


def _view(psi, bits):
    """psi with a dimension of its own for every listed bit, the highest
    first, and the dimension that each bit got."""
    n = psi.numel().bit_length() - 1
    shape, dims, at = [], {}, n
    for b in sorted(bits, reverse=True):
        shape += [2 ** (at - 1 - b), 2]
        dims[b] = len(shape) - 1
        at = b
    return psi.view(shape + [2 ** at]), dims


def _simulate(n, x0, gates):
    """The final state and the layout that virtual swaps leave."""
    l2p = list(range(n))
    psi = torch.zeros(2 ** n, dtype=torch.complex128, device=DEVICE)
    psi[x0] = 1
    open_ = {}                       # one-qubit matrices not applied yet, by physical bit

    def apply_1q(b, m):
        v = psi.view(-1, 2, 2 ** b)
        lo = v[:, 0] * complex(m[0, 0]) + v[:, 1] * complex(m[0, 1])
        v[:, 1] = v[:, 0] * complex(m[1, 0]) + v[:, 1] * complex(m[1, 1])
        v[:, 0] = lo

    def close(bits):
        for b in bits:
            if b in open_:
                apply_1q(b, open_.pop(b))

    for g in gates:
        kind = g[0]
        if kind == "swap":
            a, b = g[1]
            l2p[a], l2p[b] = l2p[b], l2p[a]
            continue
        bits = [l2p[v] for v in g[1]]
        if len(bits) == 1:
            open_[bits[0]] = _matrix(g) @ open_.get(bits[0], np.eye(2))
            continue
        close(bits)
        v, dims = _view(psi, bits)

        def part(v, *ones):
            for d, x in sorted(ones, reverse=True):
                v = v.select(d, x)
            return v

        if kind == "dense":
            k = len(bits)
            first = [dims[b] for b in reversed(bits)]       # matrix bit 0 is the last of these
            order = first + [d for d in range(v.dim()) if d not in first]
            w = v.permute(order).reshape(2 ** k, -1)
            w = (torch.from_numpy(_matrix(g)).to(DEVICE) @ w).view([v.shape[d] for d in order])
            v.copy_(w.permute([order.index(d) for d in range(v.dim())]))
        elif kind == "cx":
            a, b = dims[bits[0]], dims[bits[1]]
            lo = part(v, (a, 1), (b, 0)).clone()
            part(v, (a, 1), (b, 0)).copy_(part(v, (a, 1), (b, 1)))
            part(v, (a, 1), (b, 1)).copy_(lo)
        elif kind in ("cz", "cp"):
            ph = -1.0 if kind == "cz" else complex(math.cos(g[2][0]), math.sin(g[2][0]))
            part(v, (dims[bits[0]], 1), (dims[bits[1]], 1)).mul_(ph)
        else:                                               # rzz
            for x in (0, 1):
                for y in (0, 1):
                    a = g[2][0] / 2 * (1 if x != y else -1)
                    part(v, (dims[bits[0]], x), (dims[bits[1]], y)).mul_(complex(math.cos(a), math.sin(a)))
    close(sorted(open_))
    return psi, l2p


def _sum_bits(p, keep):
    """Sums p over every bit not in `keep`; the kept bits stay in order."""
    n = p.numel().bit_length() - 1
    for b in range(n - 1, -1, -1):
        if b not in keep:
            p = p.view(-1, 2, 2 ** b).sum(1).view(-1)
    return p


def _zz(p, a, b):
    lo, hi = min(a, b), max(a, b)
    s = _sum_bits(p, (lo, hi)).tolist()
    return s[0] - s[1] - s[2] + s[3]


def _z(p, n):
    """<Z> of every bit: marginals halve the array from the top bit down."""
    out = [0.0] * n
    for b in range(n - 1, -1, -1):
        v = p.view(2, -1)
        s = v.sum(1).tolist()
        out[b] = s[0] - s[1]
        p = v.sum(0)
    return out


def exact(case, seed):
    op, n = case["op"], case["n"]
    if op == "circuit":
        x0, gates = _circuit(case, seed)
        if _gate_flops(gates, n) > 2.0e13:                  # over about 20 seconds
            return None
        return torch.view_as_real(_simulate(n, x0, gates)[0]).reshape(-1)
    if op == "qaoa":
        edges, _, gates = _qaoa_inputs(case, seed)
        psi = _simulate(n, 0, gates)[0]
        p = psi.real.square() + psi.imag.square()
        return {"state": torch.view_as_real(psi).reshape(-1), "zz": np.array([_zz(p, a, b) for a, b in edges])}
    if op == "batch":
        out = []
        for m, gates in _batch_inputs(case, seed):
            psi = _simulate(m, 0, gates)[0]
            out += _z(psi.real.square() + psi.imag.square(), m)
        return np.array(out)
    buf, swaps, asked = _random_state(case, seed)
    p = buf.view(-1, 2).double().square().sum(1)
    del buf
    l2p = list(range(n))
    for a, b in swaps:
        l2p[a], l2p[b] = l2p[b], l2p[a]
    if op == "expect_z":
        z = _z(p, n)
        return np.array([z[l2p[b]] for b in range(n)])
    if op == "zz":
        return np.array([_zz(p, l2p[a], l2p[b]) for a, b in asked])
    bits = [l2p[b] for b in asked]                          # output index bit j is physical bit bits[j]
    kept = sorted(bits)
    p = _sum_bits(p, kept)
    v = p.view([2] * len(kept))                             # dimension i is bit kept[-1 - i]
    return v.permute([len(kept) - 1 - kept.index(b) for b in reversed(bits)]).reshape(-1)
