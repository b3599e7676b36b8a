"""The work that users of this library have it do, as timed cases.

Each case is one pass through the public entry points, as a user's program
calls them: whole circuit runs from a basis state, from widths where latency
decides to states of gigabytes; single gates on a live state; the read-outs
of a state; a batch of cut variants and their reconstruction; a qubit
relabelling; a burst of requests to the server.  ``prepare`` makes what such
a program holds before the call (circuits, states, plans of a batch, output
buffers), ``run`` makes the call, ``exact`` computes the same outputs in 64
bits with plain torch.

Circuits are the layered ones of the benchmark: U3 on every qubit with
angles uniform on [0, 2 pi), then a brick wall of CZ (or CZ / CNOT) on
neighbouring qubits; and the QFT-style one, a Fourier ladder on a random
basis state followed by such layers.
"""
import collections
import dataclasses
import math

import numpy as np
import torch

from paper_2502_11385_amd import qsv

Gate = collections.namedtuple("Gate", "name qubits params")
TWO_PI = 2.0 * math.pi
LABELS = ("0", "1", "+", "+i")
BASES = ("I", "X", "Y")


@dataclasses.dataclass
class Variant:
    width: int
    gates: list
    cut_inputs: list
    cut_outputs: list


@dataclasses.dataclass
class Sub:
    width: int
    out_qubit: list
    cut_in: list
    cut_out: list


def listed():
    return [
        # The smallest whole circuit of the benchmark: 12 qubits, depth 20.
        # One launch sequence per circuit; latency and host work count.
        {"name": "small_c64", "kind": "circuit", "n": 12, "depth": 20,
         "prec": "c64"},
        # A user who wants 64-bit amplitudes of a small, odd-sized circuit
        # (13 qubits: two tiles, the first width with more than one pass).
        {"name": "small_c128", "kind": "circuit", "n": 13, "depth": 12,
         "prec": "c128"},
        # The 20-qubit instance of the headline circuit: a state that fits
        # the last-level cache, several passes, host planning visible.
        {"name": "mid_c64", "kind": "circuit", "n": 20, "depth": 40,
         "prec": "c64"},
        # A middle-sized 64-bit run of odd width whose caller reads the
        # amplitudes themselves.
        {"name": "mid_c128", "kind": "circuit", "n": 23, "depth": 30,
         "prec": "c128"},
        # The headline workload: 30 qubits, depth 40, probabilities and the
        # marginal of the top ten qubits out of the last pass.
        {"name": "large_c64", "kind": "circuit", "n": 30, "depth": 40,
         "prec": "c64"},
        # A Fourier ladder (long runs of controlled phases) on a random
        # basis state, then ten layers, in 64 bits; a marginal is read.
        {"name": "qft_c128", "kind": "qft", "n": 26, "tail": 10,
         "prec": "c128"},
        # Interactive use: single gates of every kind on a live state, one
        # call each (1 to 5 targets, controls, diagonals).
        {"name": "gates_c64", "kind": "gates", "n": 27, "count": 24,
         "prec": "c64"},
        # Everything a user reads from a finished state: probabilities,
        # norm, a marginal, shots, the most probable outcomes, Pauli
        # expectation values.
        {"name": "readout_c64", "kind": "readout", "n": 27, "shots": 100000,
         "prec": "c64"},
        # Relabelling the qubits of a 64-bit state: a random permutation,
        # the data movement of swap insertion.
        {"name": "relabel_c128", "kind": "relabel", "n": 27, "prec": "c128"},
        # Subcircuit variants of a cut circuit in one batch: ragged widths
        # 10 to 20 and depths 10 to 60, probabilities of each.
        {"name": "batch_c64", "kind": "batch", "count": 192, "wmin": 10,
         "wmax": 20, "prec": "c64"},
        # Rebuilding the uncut distribution of a chain of three subcircuits
        # from its 19 variants' vectors.
        {"name": "cut_28", "kind": "cut", "w0": 9, "w1": 12, "w2": 9,
         "prec": "c64"},
        # A burst of requests to the server, small ones batched, wide ones
        # alone, a fifth of them in 64 bits; probability vectors come back.
        {"name": "serve_burst", "kind": "serve", "count": 40, "wmin": 8,
         "wmax": 22},
    ]


def draw(rng):
    """One more case of the same ranges, sizes spread over the whole of each
    (a width is the logarithm of the work)."""
    kind = rng.choice(["circuit", "circuit", "circuit", "qft", "gates",
                       "readout", "relabel", "batch", "cut", "serve"])
    prec = rng.choice(["c64", "c64", "c128"])
    if kind == "circuit":
        return {"kind": kind, "n": rng.randint(8, 27),
                "depth": int(round(2 ** rng.uniform(2.0, 5.9))), "prec": prec}
    if kind == "qft":
        return {"kind": kind, "n": rng.randint(10, 27),
                "tail": rng.randint(0, 10), "prec": prec}
    if kind == "gates":
        return {"kind": kind, "n": rng.randint(8, 27),
                "count": rng.randint(8, 32), "prec": prec}
    if kind == "readout":
        return {"kind": kind, "n": rng.randint(10, 27),
                "shots": int(round(2 ** rng.uniform(6.0, 18.0))),
                "prec": prec}
    if kind == "relabel":
        return {"kind": kind, "n": rng.randint(8, 27), "prec": prec}
    if kind == "batch":
        lo = rng.randint(6, 14)
        return {"kind": kind, "count": int(round(2 ** rng.uniform(3.0, 7.5))),
                "wmin": lo, "wmax": rng.randint(lo, 20), "prec": prec}
    if kind == "cut":
        return {"kind": kind, "w0": rng.randint(4, 10),
                "w1": rng.randint(4, 11), "w2": rng.randint(4, 9),
                "prec": prec}
    return {"kind": kind, "count": rng.randint(6, 48),
            "wmin": rng.randint(6, 12), "wmax": rng.randint(13, 22)}


# ------------------------------------------------------------------ inputs


def _rng(seed):
    return np.random.Generator(np.random.PCG64([int(seed), 2502]))


def _prec(case):
    return qsv.QSV_C64 if case["prec"] == "c64" else qsv.QSV_C128


def _ctype(case):
    return torch.complex64 if case["prec"] == "c64" else torch.complex128


def _layers(rng, n, depth, mixed=False):
    angles = rng.uniform(0.0, TWO_PI, size=(depth, n, 3))
    gates = []
    for layer in range(depth):
        for q in range(n):
            gates.append(Gate("u3", (q,), tuple(map(float, angles[layer, q]))))
        for a in range(layer % 2, n - 1, 2):
            name = "cx" if mixed and rng.integers(0, 2) else "cz"
            gates.append(Gate(name, (a, a + 1), ()))
    return gates


def _circuit_gates(case, seed):
    """(basis index, gates) of a whole-circuit case."""
    rng, n = _rng(seed), case["n"]
    if case["kind"] == "circuit":
        return 0, _layers(rng, n, case["depth"])
    x = int(rng.integers(0, 1 << n))
    gates = []
    for j in range(n - 1, -1, -1):
        gates.append(Gate("h", (j,), ()))
        for k in range(1, j + 1):
            gates.append(Gate("cp", (j - k, j), (math.pi / (1 << k),)))
    return x, gates + _layers(rng, n, case["tail"])


def _unitary(rng, k):
    d = 1 << k
    q, r = np.linalg.qr(rng.standard_normal((d, d)) +
                        1j * rng.standard_normal((d, d)))
    return q * (np.diagonal(r) / np.abs(np.diagonal(r)))


def _gate_calls(case, seed):
    """(targets, matrix, controls) of single-gate calls: the mix of a
    program that drives a state gate by gate, qubits drawn uniformly."""
    rng, n = _rng(seed), case["n"]
    kinds = ["u3", "cx", "cz", "u3", "rz", "two", "u3", "cp", "u3", "ccx",
             "three", "u3", "cu", "four", "u3", "cz", "five", "s", "cx"]
    out = []
    for i in range(case["count"]):
        kind = kinds[i % len(kinds)]
        q = [int(v) for v in rng.permutation(n)[:5]]
        ph = complex(np.exp(1j * rng.uniform(0.0, TWO_PI)))
        x = np.array([[0, 1], [1, 0]], dtype=complex)
        if kind == "u3":
            out.append((q[:1], _unitary(rng, 1), []))
        elif kind == "cx":
            out.append((q[:1], x, q[1:2]))
        elif kind == "ccx":
            out.append((q[:1], x, q[1:3]))
        elif kind == "cu":
            out.append((q[:1], _unitary(rng, 1), q[1:2]))
        elif kind == "cz":
            out.append((q[:1], np.diag([1, -1]).astype(complex), q[1:2]))
        elif kind == "cp":
            out.append((q[:1], np.diag([1, ph]), q[1:2]))
        elif kind == "s":
            out.append((q[:1], np.diag([1, 1j]).astype(complex), []))
        elif kind == "rz":
            out.append((q[:1], np.diag([ph.conjugate(), ph]), []))
        else:
            k = {"two": 2, "three": 3, "four": 4, "five": 5}[kind]
            out.append((q[:k], _unitary(rng, k), []))
    return out


def _random_state(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 2 + 1)
    t = torch.randn(1 << case["n"], dtype=_ctype(case), device="cuda",
                    generator=g)
    return t.div_(torch.linalg.vector_norm(t))


def _shapes(case):
    """(width, depth) of a ragged case's circuits, the same for each seed."""
    rng = _rng(case["count"] * 1024 + case["wmin"] * 32 + case["wmax"])
    return [(int(rng.integers(case["wmin"], case["wmax"] + 1)),
             int(rng.integers(10, 61))) for _ in range(case["count"])]


def _variants(case, seed):
    rng = _rng(seed)
    out = []
    for w, d in _shapes(case):
        qi = rng.choice(w, size=int(rng.integers(1, 4)), replace=False)
        qo = rng.choice(w, size=int(rng.integers(1, 4)), replace=False)
        ins = [(int(q), LABELS[int(rng.integers(0, 4))]) for q in qi]
        outs = [(int(q), BASES[int(rng.integers(0, 3))]) for q in qo]
        out.append(Variant(w, _layers(rng, w, d, mixed=True), ins, outs))
    return out


def _cut_subs(case):
    """A chain of three subcircuits, the last qubit of each cut towards the
    first qubit of the next; uncut qubits numbered as they appear."""
    w0, w1, w2 = case["w0"], case["w1"], case["w2"]
    n1 = w0 - 1            # uncut qubit on the first cut wire
    n2 = w0 + w1 - 2       # and on the second
    s0 = Sub(w0, list(range(w0 - 1)) + [-1], [-1] * w0,
             [-1] * (w0 - 1) + [0])
    s1 = Sub(w1, list(range(n1, n1 + w1 - 1)) + [-1], [0] + [-1] * (w1 - 1),
             [-1] * (w1 - 1) + [1])
    s2 = Sub(w2, list(range(n2, n2 + w2)), [1] + [-1] * (w2 - 1), [-1] * w2)
    return n2 + w2, [s0, s1, s2]


def _cut_vectors(case, seed):
    """The variants' probability vectors, one after the other."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 2 + 1)
    dt = torch.float32 if case["prec"] == "c64" else torch.float64
    parts = []
    for w, count in ((case["w0"], 3), (case["w1"], 12), (case["w2"], 4)):
        p = -torch.log(torch.rand(count, 1 << w, dtype=torch.float64,
                                  device="cuda", generator=g) + 1e-300)
        parts.append((p / p.sum(1, keepdim=True)).to(dt).reshape(-1))
    offs, at = [], 0
    for w, count in ((case["w0"], 3), (case["w1"], 12), (case["w2"], 4)):
        for _ in range(count):
            offs.append(at)
            at += 1 << w
    return torch.cat(parts), np.asarray(offs, np.uint64)


def _requests(case, seed):
    rng = _rng(seed)
    out = []
    for i, (w, d) in enumerate(_shapes(case)):
        out.append((w, i % 5 == 2, _layers(rng, w, d)))
    return out


def _readout_terms(case, seed):
    rng = _rng(seed)
    terms = []
    for weight in (2, 3, 4, 1):
        qs = rng.permutation(case["n"])[:weight]
        terms.append({int(q): "XYZ"[int(rng.integers(0, 3))] for q in qs})
    marg = [int(q) for q in rng.permutation(case["n"])[:min(8, case["n"])]]
    return terms, marg


def prepare(case, seed):
    kind, st = case["kind"], dict(case)
    stream = torch.cuda.current_stream()
    if kind in ("circuit", "qft"):
        st["basis"], gates = _circuit_gates(case, seed)
        st["circ"] = qsv.Circuit.from_gates(gates)
        st["circ"].arrays()
        n = case["n"]
        if kind == "circuit" and case["prec"] == "c64":
            st["state"] = qsv.State(n, _prec(case), stream=stream)
            dt = torch.float64 if n < 16 else torch.float32
            st["probs"] = torch.empty(1 << n, dtype=dt, device="cuda")
        else:
            st["amps"] = torch.empty(1 << n, dtype=_ctype(case),
                                     device="cuda")
            st["state"] = qsv.State(n, _prec(case), stream=stream,
                                    tensor=st["amps"])
    elif kind in ("gates", "readout", "relabel"):
        st["amps"] = _random_state(case, seed)
        st["state"] = qsv.State(case["n"], _prec(case), stream=stream,
                                tensor=st["amps"])
        if kind == "gates":
            st["calls"] = _gate_calls(case, seed)
        elif kind == "readout":
            st["terms"], st["marg"] = _readout_terms(case, seed)
            st["probs"] = torch.empty(1 << case["n"], dtype=torch.float32,
                                      device="cuda")
            st["seed"] = int(seed)
        else:
            st["perm"] = [int(q) for q in _rng(seed).permutation(case["n"])]
    elif kind == "batch":
        st["batch"] = qsv.Batch(_variants(case, seed), prec=_prec(case),
                                stream=stream,
                                out_fp64=case["prec"] == "c128")
        st["out"] = st["batch"].output()
    elif kind == "cut":
        n, subs = _cut_subs(case)
        st["spec"] = qsv.CutSpec(n, 2, subs)
        st["vectors"], st["offsets"] = _cut_vectors(case, seed)
        st["work"] = torch.empty(max(1, st["spec"].workspace_bytes()),
                                 dtype=torch.uint8, device="cuda")
        st["out"] = torch.empty(1 << n, dtype=torch.float64, device="cuda")
        st["stream"] = stream
    else:
        st["requests"] = [
            (w, qsv.QSV_C128 if wide else qsv.QSV_C64,
             qsv.Circuit.from_gates(gates))
            for w, wide, gates in _requests(case, seed)]
        st["server"] = qsv.Server()
    return st


# -------------------------------------------------------------------- runs


def run(st):
    kind = st["kind"]
    if kind in ("circuit", "qft"):
        s = st["state"]
        s.init_basis(st["basis"])
        if "amps" not in st:
            if st["n"] < 16:        # a small circuit: FP64 probabilities
                s.apply_fused(st["circ"])
                s.probabilities_into(st["probs"].data_ptr(), True)
                return st["probs"]
            marg, _ = s.apply_fused_outputs(
                st["circ"], probs_ptr=st["probs"].data_ptr(),
                marg_qubits=list(range(st["n"] - 10, st["n"])))
            return {"probs": st["probs"], "marginal": marg}
        s.apply_fused(st["circ"])
        if kind == "qft":
            top = list(range(st["n"] - 10, st["n"]))
            return {"amps": st["amps"], "marginal": s.marginal(top)}
        return st["amps"]
    if kind == "gates":
        for targets, matrix, controls in st["calls"]:
            st["state"].apply_gate(targets, matrix, controls)
        return st["amps"]
    if kind == "readout":
        s = st["state"]
        s.probabilities_into(st["probs"].data_ptr(), False)
        idx, p = s.top_k(64)
        return {"probs": st["probs"], "norm": s.norm(),
                "marginal": s.marginal(st["marg"]),
                "shots": s.sample(st["shots"], st["seed"]),
                "top_index": idx, "top_p": p,
                "expectation": s.expectation(st["terms"])}
    if kind == "relabel":
        st["state"].permute_qubits(st["perm"])
        return st["amps"]
    if kind == "batch":
        st["batch"].launch(st["out"])
        return st["out"]
    if kind == "cut":
        qsv.cut_reconstruct(st["spec"], st["vectors"], st["offsets"],
                            st["out"], st["work"], st["stream"])
        return st["out"]
    srv = st["server"]
    tickets = [srv.submit(w, circ, prec) for w, prec, circ in st["requests"]]
    out = []
    for t in tickets:
        out.append(srv.wait(t)[0])
        srv.release(t)
    return out


def _circuit_work(n, gates):
    """Flops of a circuit gate by gate: a complex 2x2 row (14) on every
    amplitude for a dense gate, a complex product (6) on the quarter of the
    amplitudes that a controlled phase changes; none for CZ and CNOT."""
    flops = 0.0
    for g in gates:
        if g.name in ("u3", "h"):
            flops += 14.0 * 2.0 ** n
        elif g.name == "cp":
            flops += 6.0 * 2.0 ** (n - 2)
    return flops


def work(case):
    kind = case["kind"]
    b = 8 if case.get("prec") == "c64" else 16
    if kind in ("circuit", "qft"):
        n = case["n"]
        _, gates = _circuit_gates(case, 0)
        out = (8 if n < 16 else 4) if kind == "circuit" and b == 8 else b
        return {"bytes": float(out << n), "flops": _circuit_work(n, gates)}
    if kind == "gates":
        nbytes = flops = 0.0
        for targets, matrix, controls in _gate_calls(case, 0):
            k, c = len(targets), len(controls)
            part = 2.0 ** (case["n"] - c)
            m = np.asarray(matrix)
            if np.count_nonzero(m - np.diag(np.diagonal(m))) == 0:
                part *= 0.5 if m[0, 0] == 1 else 1.0
                flops += 6.0 * part
            else:
                flops += (8.0 * 2 ** k - 2.0) * part
            nbytes += 2.0 * b * part
        return {"bytes": nbytes, "flops": flops}
    if kind == "readout":
        # one read of the state for each quantity that a user may ask for
        # alone: probabilities, norm, marginal, shots, top, four terms
        amps = 2.0 ** case["n"]
        return {"bytes": amps * (b * 9.0 + 4.0) + 8.0 * case["shots"],
                "flops": amps * 40.0}
    if kind == "relabel":
        return {"bytes": 2.0 * b * 2.0 ** case["n"], "flops": 0.0}
    if kind == "cut":
        n = case["w0"] + case["w1"] + case["w2"] - 2
        return {"bytes": 8.0 * 2.0 ** n, "flops": 2.0 * 16 * 2.0 ** n}
    if kind == "batch":
        flops = nbytes = 0.0
        for v in _variants(case, 0):
            flops += _circuit_work(v.width, v.gates)
            nbytes += (b // 2) * 2.0 ** v.width
        return {"bytes": nbytes, "flops": flops}
    flops = nbytes = 0.0
    for w, wide, gates in _requests(case, 0):
        flops += _circuit_work(w, gates)
        nbytes += (8 if wide else 4) * 2.0 ** w
    return {"bytes": nbytes, "flops": flops}


# ------------------------------------------------- the same in 64 bits


def _matrix(g):
    """(targets, 2x2 matrix, controls) of a named gate, OpenQASM's U3."""
    r = math.sqrt(0.5)
    if g.name == "u3":
        th, ph, la = g.params
        c, s = math.cos(th / 2), math.sin(th / 2)
        e = lambda a: complex(math.cos(a), math.sin(a))  # noqa: E731
        return g.qubits, [[c, -e(la) * s], [e(ph) * s, e(ph + la) * c]], ()
    if g.name == "h":
        return g.qubits, [[r, r], [r, -r]], ()
    if g.name == "sdg":
        return g.qubits, [[1, 0], [0, -1j]], ()
    if g.name == "s":
        return g.qubits, [[1, 0], [0, 1j]], ()
    if g.name == "x":
        return g.qubits, [[0, 1], [1, 0]], ()
    if g.name == "cx":
        return g.qubits[1:], [[0, 1], [1, 0]], g.qubits[:1]
    if g.name == "cz":
        return g.qubits[1:], [[1, 0], [0, -1]], g.qubits[:1]
    lam = g.params[0]
    return (g.qubits[1:], [[1, 0], [0, complex(math.cos(lam), math.sin(lam))]],
            g.qubits[:1])


def _apply(psi, n, targets, matrix, controls):
    """psi <- matrix on targets where the controls are 1 (in place)."""
    qs = sorted((*targets, *controls), reverse=True)
    shape, hi = [], n
    for q in qs:
        shape += [1 << (hi - q - 1), 2]
        hi = q
    v = psi.view(shape + [1 << hi])
    at = [slice(None)] * v.dim()
    for c in controls:
        at[2 * qs.index(c) + 1] = 1
    k = len(targets)

    def part(r):
        w = list(at)
        for j, t in enumerate(targets):
            w[2 * qs.index(t) + 1] = r >> j & 1
        return v[tuple(w)]

    m = [[complex(x) for x in row] for row in np.asarray(matrix)]
    if all(m[r][c] == 0 for r in range(1 << k) for c in range(1 << k)
           if r != c):
        for r in range(1 << k):
            if m[r][r] != 1:
                part(r).mul_(m[r][r])
        return
    old = [part(r).clone() for r in range(1 << k)]
    for r in range(1 << k):
        acc = old[0] * m[r][0]
        for c in range(1, 1 << k):
            acc.add_(old[c], alpha=m[r][c])
        part(r).copy_(acc)


def _simulate(n, basis, gates):
    psi = torch.zeros(1 << n, dtype=torch.complex128, device="cuda")
    psi[basis] = 1
    for g in gates:
        t, m, c = _matrix(g)
        _apply(psi, n, t, m, c)
    return psi


def _probs(psi):
    return psi.real.square() + psi.imag.square()


def _marginal(p, n, qubits):
    """P[j] over the qubits' bits, qubits[0] the least significant."""
    keep = [n - 1 - q for q in reversed(qubits)]
    lost = [a for a in range(n) if a not in keep]
    t = p.view([2] * n).permute(keep + lost).reshape(1 << len(qubits), -1)
    return t.sum(1).cpu().numpy()


def exact(case, seed):
    kind = case["kind"]
    if kind in ("circuit", "qft"):
        n = case["n"]
        basis, gates = _circuit_gates(case, seed)
        if n > 27 or len(gates) * 2.0 ** n > 2.0 ** 37.5:
            return None
        psi = _simulate(n, basis, gates)
        top = list(range(n - 10, n))
        if kind == "qft":
            return {"amps": psi, "marginal": _marginal(_probs(psi), n, top)}
        if case["prec"] == "c128":
            return psi
        p = _probs(psi)
        if n < 16:
            return p
        return {"probs": p, "marginal": _marginal(p, n, top)}
    if kind == "gates":
        psi = _random_state(case, seed).to(torch.complex128)
        for targets, matrix, controls in _gate_calls(case, seed):
            _apply(psi, case["n"], targets, matrix, controls)
        return psi
    if kind == "readout":
        n = case["n"]
        psi = _random_state(case, seed).to(torch.complex128)
        p = _probs(psi)
        terms, marg = _readout_terms(case, seed)
        values = []
        for term in terms:
            phi = psi.clone()
            for q, lab in term.items():
                m = {"X": [[0, 1], [1, 0]], "Y": [[0, -1j], [1j, 0]],
                     "Z": [[1, 0], [0, -1]]}[lab]
                _apply(phi, n, [q], m, [])
            values.append(float((psi.conj() * phi).real.sum()))
        top = torch.topk(p, 64).values
        return {"probs": p, "norm": float(p.sum()), "shots": None,
                "marginal": _marginal(p, n, marg), "top_index": None,
                "top_p": top.cpu().numpy(), "expectation": np.array(values)}
    if kind == "relabel":
        n = case["n"]
        psi = _random_state(case, seed).to(torch.complex128)
        perm = [int(q) for q in _rng(seed).permutation(n)]
        at = torch.arange(1 << n, device="cuda")
        src = torch.zeros_like(at)
        for q, to in enumerate(perm):       # bit perm[q] was bit q
            src |= (at >> to & 1) << q
        return psi[src]
    if kind == "cut":
        return _exact_cut(case, seed)
    if kind == "batch":
        variants = _variants(case, seed)
        if sum(len(v.gates) for v in variants) > 160000:
            return None
        out = []
        for v in variants:
            pre, post = [], []
            for q, lab in v.cut_inputs:
                pre += [Gate(name, (q,), ()) for name in
                        {"0": "", "1": "x", "+": "h", "+i": "hs"}[lab]]
            for q, basis in v.cut_outputs:
                if basis == "Y":
                    post.append(Gate("sdg", (q,), ()))
                if basis != "I":
                    post.append(Gate("h", (q,), ()))
            out.append(_probs(_simulate(v.width, 0, pre + v.gates + post)))
        return torch.cat(out)
    return [_probs(_simulate(w, 0, gates)).cpu().numpy()
            for w, _, gates in _requests(case, seed)]


def _exact_cut(case, seed):
    """(1/2)^2 times the sum, over four terms for each of the two cuts, of
    the product of the subcircuits' term vectors."""
    vec, _ = _cut_vectors(case, seed)
    vec = vec.to(torch.float64)
    w0, w1, w2 = case["w0"], case["w1"], case["w2"]
    a = vec[:3 << w0].view(3, 1 << w0)
    b = vec[3 << w0:(3 << w0) + (12 << w1)].view(3, 4, 1 << w1)
    c = vec[(3 << w0) + (12 << w1):].view(4, 1 << w2)

    def upstream(v, t):       # measured qubit is the most significant bit
        v = v[(0, 0, 1, 2)[t]]
        lo, hi = v.chunk(2, dim=-1)
        return (2 * lo, 2 * hi, lo - hi, lo - hi)[t]

    def downstream(v, t):
        return v[t] if t < 2 else 2 * v[t] - v[0] - v[1]

    n0, n1, n2 = 1 << (w0 - 1), 1 << (w1 - 1), 1 << w2
    out = torch.zeros(n2, n1 * n0, dtype=torch.float64, device="cuda")
    for t1 in range(4):
        mid = torch.zeros(n1 * n0, dtype=torch.float64, device="cuda")
        for t0 in range(4):
            m = torch.stack([upstream(b[:, i], t1) for i in range(4)])
            mid += torch.outer(downstream(m, t0), upstream(a, t0)).view(-1)
        out.addcmul_(downstream(c, t1).view(-1, 1), mid.view(1, -1),
                     value=0.25)
    return out.view(-1)
