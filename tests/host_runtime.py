"""The library on a fake HIP runtime (tests/fake_hip.cpp), one check per run:
python host_runtime.py FAKE_LIBRARY CHECK.  The fake's symbols have to come
before the real runtime's, so a check needs a process of its own."""
import ctypes
import os
import re
import struct
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

CALLBACK = ctypes.CFUNCTYPE(None, ctypes.c_int, ctypes.c_char_p, ctypes.c_uint64, ctypes.c_uint64,
                            ctypes.POINTER(ctypes.c_void_p))
RC_1Q_LANE, RC_1Q_REG, RC_SHEAR_REG = 5, 23, 38    # operation codes (devprog.hpp)


def argument(args, i, ctype):
    return ctypes.cast(args[i], ctypes.POINTER(ctype))[0]


def tile_pass(args, prec):
    """A register tile pass: the factor of its store and its operations as
    (code, entries)."""
    hdr = ctypes.string_at(argument(args, 1, ctypes.c_void_p), 240)
    ops = argument(args, 2, ctypes.c_void_p)
    nops, op0 = struct.unpack("2i", hdr[12:20])
    size = 64 if prec == 0 else 128
    recs = []
    for i in range(nops):
        r = ctypes.string_at(ops + 64 * op0 + size * i, size)
        k = struct.unpack("8f", r[24:56]) if prec == 0 else struct.unpack("8d", r[24:56] + r[64:96])
        recs.append((struct.unpack("i", r[:4])[0], [complex(k[2 * e], k[2 * e + 1]) for e in range(4)]))
    return struct.unpack("d", hdr[232:240])[0], recs


def sweep(n, depth, seed=0.1):
    g = []
    for d in range(depth):
        for b in range(n):
            g += [("ry", (b,), (seed + 0.01 * b + d,)), ("rz", (b,), (seed - 0.02 * b + d,))]
        g += [("cz", (b, b + 1)) for b in range(d & 1, n - 1, 2)]
    return g


class Fake:
    def __init__(self, path):
        self.lib = ctypes.CDLL(path, ctypes.RTLD_GLOBAL)
        self.lib.fake_stream.restype = ctypes.c_void_p
        self.lib.fake_capture.argtypes = [ctypes.c_void_p, ctypes.c_int]
        self.on_launch = lambda index, kernel, grid, block, args: None
        self._cb = CALLBACK(lambda i, k, g, b, a: self.on_launch(i, k.decode(), g, b, a))
        self.lib.fake_on_launch(self._cb)


def state(q, n, prec, stream=None):
    h = ctypes.c_void_p()
    q.check(q.lib().qops_create(n, prec, None, 0, stream, ctypes.byref(h)))
    return h


def deep_layers(n, busy, layers, gate):
    g = []
    for _ in range(layers):
        g += [(gate[0], (b,), gate[1]) for b in range(busy)]
        g += [("cz", (b, b + 1)) for b in range(busy - 1)]
    return g


def check_growth(fake, q):
    """A chain of 2x2s keeps the amplitudes in range: what its operations have
    not applied yet (the next full 2x2 or the pass's store does) stays above
    2^-17 on each bit, 2^-66 in all."""
    seen = []

    def on_launch(i, kernel, grid, block, args):
        if "tile_pass_kernel" in kernel:
            seen.append(tile_pass(args, prec))
    fake.on_launch = on_launch
    for prec in (0, 1):
        for n, busy, up in ((10, 10, 0), (11, 11, 0), (12, 12, 0), (13, 4, 7), (20, 4, 0)):
            for gate in (("h", ()), ("rx", (1.5707963267948966,)), ("u3", (1.2, 0.3, 2.2))):
                seen.clear()
                p = q.Plan(n, deep_layers(n, busy, 400, gate), precision=prec, tile_upper=up)
                h = state(q, n, prec)
                q.check(q.lib().qops_run_plan(h, p.handle))
                assert seen
                for scale, recs in seen:
                    assert scale >= 2.0 ** -66, (prec, n, gate, scale)
                    for code, k in recs:
                        if RC_1Q_LANE <= code < RC_1Q_LANE + 3 or RC_1Q_REG <= code < RC_SHEAR_REG:
                            assert max(abs(x) for x in k) >= 2.0 ** -17, (prec, n, gate, code, k)
                q.lib().qops_destroy(h)


def check_batch_order(fake, q):
    """In a batch's stream order and in its graph a circuit's pass p ends
    before its pass p + 1 begins, and every pass before the <Z> reduction."""
    runs = []

    def on_launch(i, kernel, grid, block, args):
        if not runs or (runs[-1] and runs[-1][-1][2] == "z"):
            runs.append([])                      # the eager run, then the capture
        if "tile_pass_kernel" in kernel:
            items = argument(args, 5, ctypes.c_void_p)
            count = argument(args, 4, ctypes.c_uint64)
            circs = {struct.unpack("2i", ctypes.string_at(items + 8 * j, 8))[0] for j in range(count)}
            runs[-1].append((i, circs, argument(args, 7, ctypes.c_int32)))
        elif "batch_zfinal" in kernel:
            runs[-1].append((i, None, "z"))
    fake.on_launch = on_launch
    dense = [("dense", (0, 1), (), (), [[1, 0, 0, 0], [0, 0, 1, 0], [0, 1, 0, 0], [0, 0, 0, 1]])]
    for prec in (0, 1):
        for circs in ([(13, sweep(13, d)) for d in (24, 64, 128)], [(12, sweep(12, 160)), (13, sweep(13, 40))],
                      [(n, sweep(n, d)) for n, d in ((8, 5), (10, 300), (11, 200), (12, 3), (12, 130), (13, 70), (15, 9))] +
                      [(11, sweep(11, 2) + dense)]):
            runs.clear()
            b = q.Batch(circs, precision=prec)
            assert len(runs) == 2
            for run in runs:
                last = {}
                for i, cs, step in run:
                    if step == "z":
                        assert all(fake.lib.fake_ordered(j, i) for j, c, s in run if s != "z")
                        continue
                    for c in cs:
                        assert step == (last[c][1] + 1 if c in last else 0), (prec, c, step)
                        assert c not in last or fake.lib.fake_ordered(last[c][0], i), (prec, c, step)
                        last[c] = (i, step)
                assert last
            b.close()


def check_batch_update(fake, q):
    """An update that changes a circuit's plan is refused as often as it is
    asked for, copies nothing out of its block, and leaves the batch usable."""
    def refused(b, gates):
        for _ in range(3):
            try:
                b.update(gates)
            except q.QopsError as e:
                assert e.code == -7, e          # QOPS_BAD_STATE
            else:
                raise AssertionError("accepted")

    def circuit(n, a, b):
        return [("ry", (0,), (a,)), ("ry", (0,), (b,))] + sweep(n, 3)[2:] + [("ry", (n - 1,), (a,)), ("ry", (n - 1,), (b,))]
    for prec in (0, 1):
        for ns in ((9,), (12,), (15,), (8, 11, 16)):
            def batch(a, b):
                return [circuit(n, a, b) for n in ns]
            for first, other in (((0.4, 0.2), (0.7, -0.7)), ((0.7, -0.7), (0.4, 0.2))):
                b = q.Batch(list(zip(ns, batch(*first))), precision=prec)
                refused(b, batch(*other))
                # the last circuit alone does not fit
                refused(b, batch(*first)[:-1] + batch(*other)[-1:])
                b.update(batch(*first))
                b.close()
    assert fake.lib.fake_bad_copies() == 0


def check_marginal_launches(fake, q):
    """Marginals over many bits of the largest states launch (a dispatch takes
    fewer than 2^32 work-items), also when every marginal bit is a high one."""
    import numpy as np
    launched = []
    fake.on_launch = lambda i, kernel, grid, block, args: launched.append((kernel, grid))
    for n, prec, m in ((32, 1, 24), (33, 0, 24), (33, 1, 24), (33, 1, 25), (34, 0, 25), (34, 1, 25), (34, 0, 12),
                       (30, 0, 21), (20, 0, 8)):
        h = ctypes.c_void_p()
        # a borrowed state that no kernel here reads
        q.check(q.lib().qops_create(n, prec, 4096, 16 << n, None, ctypes.byref(h)))
        out = np.zeros(1 << m)
        for qubits in (range(n - m, n), range(m)):
            launched.clear()
            q.check(q.lib().qops_probabilities(h, (ctypes.c_int32 * m)(*qubits), m,
                                               out.ctypes.data_as(ctypes.POINTER(ctypes.c_double))))
            assert any("probs_kernel" in k for k, g in launched), (n, prec, m)
        q.lib().qops_destroy(h)


def check_tile_shapes(fake, q):
    """Every register tile pass is launched with the kernel of its tile: 6 + R
    + W bits, no more than the state has."""
    def on_launch(i, kernel, grid, block, args):
        m = re.search(r"tile_pass_kernelI[fd]Li(\d)ELi(\d)E", kernel)
        if not m:
            return
        bits = 6 + int(m.group(1)) + int(m.group(2))
        hdr = argument(args, 1, ctypes.c_void_p)
        items = argument(args, 5, ctypes.c_void_p)
        at = set()
        if items:
            circs = argument(args, 6, ctypes.c_void_p)
            for j in range(argument(args, 4, ctypes.c_uint64)):
                c = struct.unpack("2i", ctypes.string_at(items + 8 * j, 8))[0]
                at.add(struct.unpack("i", ctypes.string_at(circs + 40 * c + 16, 4))[0] + argument(args, 7, ctypes.c_int32))
        for k in at or {0}:
            n, tile = struct.unpack("2i", ctypes.string_at(hdr + 240 * k, 8))
            shapes.append((n, tile, bits))
    fake.on_launch = on_launch
    shapes = []
    for prec in (0, 1):
        for small in (5, 8, 9, 10, 0):
            for bits in (0, 10, 12):
                q.Batch([(n, sweep(n, 2)) for n in range(1, 16)], precision=prec, small_max_n=small, tile_bits=bits).close()
        for n in (*range(1, 15), 18, 20, 22, 23):
            for up in range(0, 9):
                p = q.Plan(n, sweep(n, 2), precision=prec, tile_upper=up)
                h = state(q, n, prec)
                q.check(q.lib().qops_run_plan(h, p.handle))
                q.lib().qops_destroy(h)
    assert shapes
    wrong = {x for x in shapes if not (x[2] == x[1] <= x[0])}
    assert not wrong, wrong


def check_capture(fake, q):
    """While the handle's stream is captured, in every mode, a gate list is
    refused without a call that breaks the capture, and a plan that has run
    before launches its passes."""
    s = ctypes.c_void_p(fake.lib.fake_stream())
    count = []
    fake.on_launch = lambda *a: count.append(a[1])
    h = state(q, 14, 0, s)
    gates = sweep(14, 3)
    ga = q.GateArray(gates)
    p = q.Plan(14, gates, precision=0)
    q.check(q.lib().qops_run_plan(h, p.handle))
    passes = len(count)
    for mode in (0, 1, 2):
        fake.lib.fake_capture(s, mode)
        blocks = fake.lib.fake_blocks()
        assert q.lib().qops_apply(h, ga.ptr(), ga.n, None) == -6          # QOPS_HIP_ERROR
        assert fake.lib.fake_blocks() == blocks and fake.lib.hipGetLastError() == 0
        count.clear()
        q.check(q.lib().qops_run_plan(h, p.handle))
        assert len(count) == passes
        fake.lib.fake_capture(s, -1)
    q.check(q.lib().qops_apply(h, ga.ptr(), ga.n, None))
    q.lib().qops_destroy(h)


if __name__ == "__main__":
    f = Fake(sys.argv[1])
    import paper_2410_09326_amd._binding as qops
    globals()["check_" + sys.argv[2]](f, qops)
    print("ok", sys.argv[2], flush=True)
