"""Workloads by which the speed of this library is followed.

Each case is one call, or one short sequence of calls, that a program using the
library makes again and again: circuits of the sizes and shapes of the
benchmark and the tests applied through each planner, single gates, the
read-outs of one state, and batches of small circuits.  ``listed`` names fixed
ones, ``draw`` takes others of the same ranges (6 to 30 qubits, both
precisions, odd sizes among them).

kind      what one pass is
circuit   reset, then one circuit; the amplitudes
step      reset, one circuit, one 6-bit exchange, then the marginal of ten qubits;
          amplitudes and marginal (the benchmark's step, whose other read-outs
          are the readout kind)
gate      one gate on a state the program holds; the amplitudes
readout   a marginal, Z strings and shots of one state in one call
energy    expectation values of all terms of a spin Hamiltonian
batch     many variational circuits with new angles; their Z expectation values
"""
import math
from collections import namedtuple

import numpy as np
import torch

import paper_2511_14664_amd as sv
from paper_2511_14664_amd import _binding as B

Gate = namedtuple("Gate", "name targets controls params matrix", defaults=((), (), None))
MODES = {"plain": B.SV_PLAN_PLAIN, "greedy": B.SV_PLAN_GREEDY, "passes": B.SV_PLAN_PASSES}
PRECISIONS = {"native": B.SV_PREC_NATIVE, "split": B.SV_PREC_BF16X6}
AMP = {"c64": 8, "c128": 16}


def listed():
    return [
        # one entangling gate on a small register: a program that builds its state gate by gate
        {"name": "gate-10q-c64", "kind": "gate", "n": 10, "dtype": "c64", "targets": 1, "controls": 1},
        # a variational ansatz with the wrapper's defaults (one sweep per gate)
        {"name": "hea-11q-c64-plain", "kind": "circuit", "family": "hea", "n": 11, "layers": 8, "dtype": "c64",
         "mode": "plain", "precision": "native"},
        # the benchmark's 12-qubit complex128 circuit (360 gates), fused
        {"name": "layered-12q-c128-greedy", "kind": "circuit", "family": "layered", "n": 12, "layers": 20,
         "dtype": "c128", "mode": "greedy", "precision": "native"},
        # bandwidth of gate-by-gate application on a state far beyond the caches
        {"name": "layered-27q-c64-plain", "kind": "circuit", "family": "layered", "n": 27, "layers": 1, "dtype": "c64",
         "mode": "plain", "precision": "native"},
        # the fused default plan at an ordinary size
        {"name": "layered-25q-c64-greedy", "kind": "circuit", "family": "layered", "n": 25, "layers": 20,
         "dtype": "c64", "mode": "greedy", "precision": "native"},
        # the benchmark's step at its size and options
        {"name": "step-28q-c64-passes", "kind": "step", "family": "layered", "n": 28, "layers": 20, "dtype": "c64",
         "mode": "passes", "precision": "split"},
        # the same kind of circuit in double precision
        {"name": "layered-26q-c128-passes", "kind": "circuit", "family": "layered", "n": 26, "layers": 20,
         "dtype": "c128", "mode": "passes", "precision": "native"},
        # a Fourier transform of a product state: long runs of controlled phases, as in phase estimation
        {"name": "qft-29q-c64-passes", "kind": "circuit", "family": "qft", "n": 29, "layers": 1, "dtype": "c64",
         "mode": "passes", "precision": "split"},
        # random two-qubit unitaries on the largest state here
        {"name": "su4-30q-c64-passes", "kind": "circuit", "family": "su4", "n": 30, "layers": 6, "dtype": "c64",
         "mode": "passes", "precision": "split"},
        # the benchmark's read-out of one 28-qubit state
        {"name": "readout-28q-c64", "kind": "readout", "n": 28, "dtype": "c64", "bins": 10, "where": "high",
         "terms": 32, "shots": 1000},
        # energy of the transverse-field Ising model on a periodic triangular lattice
        {"name": "energy-24q-c128", "kind": "energy", "n": 24, "dtype": "c128"},
        # a parameter sweep over ansatz circuits of uneven width
        {"name": "batch-128-c64", "kind": "batch", "count": 128, "qmin": 10, "qmax": 21, "layers": 8, "dtype": "c64"},
    ]


def draw(rng):
    kind = rng.choice(["circuit", "circuit", "circuit", "step", "gate", "readout", "energy", "batch"])
    dtype = rng.choice(["c64", "c128"])
    if kind in ("circuit", "step"):
        mode = rng.choice(["plain", "greedy", "passes"]) if kind == "circuit" else "passes"
        family = rng.choice(["layered", "su4", "hea", "qft", "tfim", "rcs"]) if kind == "circuit" else "layered"
        top = 28 if dtype == "c64" else 27
        n = rng.randint(18, top) if kind == "step" else rng.randint(6, top - (2 if mode == "plain" else 0))
        if family == "tfim":
            n = 3 * max(3, n // 3)
        most = 20 if n <= 25 else 8
        if mode == "plain":
            most = 20 if n <= 18 else 4 if n <= 23 else 1
        return {"kind": kind, "family": family, "n": n, "layers": rng.randint(1, most), "dtype": dtype, "mode": mode,
                "precision": "split" if dtype == "c64" and rng.random() < 0.7 else "native"}
    if kind == "gate":
        return {"kind": kind, "n": rng.randint(6, 29 if dtype == "c64" else 28), "dtype": dtype,
                "targets": rng.randint(1, 3), "controls": rng.randint(0, 2)}
    if kind == "readout":
        n = rng.randint(14, 29 if dtype == "c64" else 28)
        return {"kind": kind, "n": n, "dtype": dtype, "bins": rng.randint(1, 12),
                "where": rng.choice(["low", "high", "any"]), "terms": rng.randint(1, 40),
                "shots": int(round(10 ** rng.uniform(1, 4)))}
    if kind == "energy":
        return {"kind": kind, "n": 3 * rng.randint(3, 8 if dtype == "c128" else 9), "dtype": dtype}
    qmin = rng.randint(6, 14)
    return {"kind": "batch", "count": int(round(2 ** rng.uniform(2, 6.5))), "qmin": qmin,
            "qmax": rng.randint(qmin, 20), "layers": rng.randint(1, 8), "dtype": dtype}


# --- inputs ---------------------------------------------------------------


def _angles(rng, k):
    return tuple(float(x) for x in rng.uniform(0.0, 2.0 * math.pi, size=k))


def _pairs(rng, n):
    p = [int(x) for x in rng.permutation(n)]
    return [(p[2 * i], p[2 * i + 1]) for i in range(n // 2)]


def _haar(rng, d):
    q, r = np.linalg.qr(rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d)))
    return q * (np.diag(r) / np.abs(np.diag(r)))


def _bonds(n):
    """Bonds of a periodic triangular lattice of 3 x n/3 sites."""
    cols = n // 3
    return [(r * cols + c, ((r + dr) % 3) * cols + (c + dc) % cols)
            for r in range(3) for c in range(cols) for dr, dc in ((0, 1), (1, 0), (1, 1))]


def _circuit(family, n, layers, rng):
    g = []
    if family == "qft":
        for _ in range(layers):
            g += [Gate("u3", (q,), (), _angles(rng, 3)) for q in range(n)]
            for t in reversed(range(n)):
                g.append(Gate("h", (t,)))
                g += [Gate("p", (t,), (t - d,), (math.pi / (1 << d),)) for d in range(1, t + 1)]
        return g
    if family in ("rcs", "tfim"):
        g += [Gate("h", (q,)) for q in range(n)]
    if family == "rcs":
        for _ in range(3 * n * layers):
            a, b = (int(x) for x in rng.choice(n, size=2, replace=False))
            kind = ("z", "h", "rx", "ry", "rz")[0 if rng.random() < 0.25 else int(rng.integers(1, 5))]
            if kind == "z":
                g.append(Gate("z", (b,), (a,)))
            else:
                g.append(Gate(kind, (a,), (), _angles(rng, 1) if kind != "h" else ()))
        return g
    theta, phi = _angles(rng, 2)
    for _ in range(layers):
        if family in ("layered", "su4"):
            g += [Gate("u3", (q,), (), _angles(rng, 3)) for q in range(n)]
            for a, b in _pairs(rng, n):
                if family == "su4":
                    g.append(Gate("matrix", (a, b), (), (), _haar(rng, 4)))
                else:
                    g.append(Gate(("x", "z")[int(rng.integers(0, 2))], (b,), (a,)))
        elif family == "hea":
            for q in range(n):
                g += [Gate("ry", (q,), (), _angles(rng, 1)), Gate("rz", (q,), (), _angles(rng, 1))]
            g += [Gate("x", (q + 1,), (q,)) for q in range(n - 1)]
        else:  # tfim: one Trotter step
            for a, b in _bonds(n):
                g += [Gate("x", (b,), (a,)), Gate("rz", (b,), (), (theta,)), Gate("x", (b,), (a,))]
            g += [Gate("rx", (q,), (), (phi,)) for q in range(n)]
    return g


def _random_state(n, dtype, seed):
    """A normalised random state on the GPU, in the precision it is held in."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    real = torch.float32 if dtype == "c64" else torch.float64
    x = torch.randn((1 << n, 2), generator=gen, device="cuda", dtype=real)
    x /= math.sqrt(float(torch.linalg.vector_norm(x, dtype=torch.float64)) ** 2)
    return torch.view_as_complex(x)


def _z_terms(n, count, rng):
    terms = []
    for _ in range(count):
        zs = set(int(x) for x in rng.choice(n, size=min(n, int(rng.integers(1, 4))), replace=False))
        terms.append("".join("Z" if q in zs else "I" for q in range(n)))
    return terms


def _ising_terms(n):
    terms = ["".join("Z" if q in (a, b) else "I" for q in range(n)) for a, b in _bonds(n)]
    return terms + ["".join("X" if q == s else "I" for q in range(n)) for s in range(n)]


def _inputs(case, seed):
    """Everything of a case that is drawn from the seed, as plain data."""
    rng = np.random.default_rng(seed)
    kind, n = case["kind"], case.get("n")
    if kind in ("circuit", "step"):
        d = {"gates": _circuit(case["family"], n, case["layers"], rng)}
        if kind == "step":
            d["qubits"] = list(range(n - 10, n))
        return d
    if kind == "gate":
        qs = [int(x) for x in rng.choice(n, size=case["targets"] + case["controls"], replace=False)]
        return {"u": _haar(rng, 1 << case["targets"]), "targets": qs[:case["targets"]],
                "controls": qs[case["targets"]:]}
    if kind == "readout":
        # bins: the lowest qubits, the highest, or any
        m = min(case["bins"], n)
        qubits = {"low": list(range(m)), "high": list(range(n - m, n)),
                  "any": [int(x) for x in rng.choice(n, size=m, replace=False)]}
        return {"qubits": qubits[case["where"]], "terms": _z_terms(n, case["terms"], rng),
                "uniforms": rng.random(case["shots"])}
    if kind == "energy":
        return {"terms": _ising_terms(n)}
    qs = [case["qmin"] + i % (case["qmax"] - case["qmin"] + 1) for i in range(case["count"])]
    return {"qs": qs, "gates": [_circuit("hea", q, case["layers"], rng) for q in qs],
            "masks": [[1 << i for i in range(q)] + [3 << i for i in range(q - 1)] for q in qs]}


class _BatchHandle:
    """A batch with its marshalled circuits, released with the object."""

    def __init__(self, dtype, batch):
        self.batch = batch
        self.handle = B.sv_batch_create(dtype, batch)

    def __del__(self):
        if getattr(self, "handle", None):
            B.sv_batch_destroy(self.handle)
            self.handle = None


def prepare(case, seed):
    kind, d = case["kind"], _inputs(case, seed)
    dtype = B.SV_C64 if case["dtype"] == "c64" else B.SV_C128
    if kind == "batch":
        b = _BatchHandle(dtype, B.Batch([B.Circuit(g) for g in d["gates"]], d["qs"], d["masks"]))
        # the configuration that the tuner picks for such batches
        B.sv_batch_set_config(b.handle, 13 if case["dtype"] == "c64" else 12, 2, 2)
        return {"case": case, "batch": b}
    s = {"case": case, "sv": sv.StateVector(case["n"], dtype), **d}
    s["amps"] = s["sv"].buffer.view(torch.complex64 if case["dtype"] == "c64" else torch.complex128)
    if kind in ("circuit", "step"):
        s["circuit"] = B.Circuit(d["gates"])
        # the benchmark's options: the order search pays where a circuit's structure is run again and again
        s["opts"] = B.make_opts(MODES[case["mode"]], 5, PRECISIONS[case["precision"]],
                                pass_orders=64 if kind == "step" else 0)
    else:
        s["amps"].copy_(_random_state(case["n"], case["dtype"], seed))
    return s


def run(state):
    kind = state["case"]["kind"]
    if kind == "batch":
        b = state["batch"]
        values = B.sv_batch_run(b.handle, b.batch, b.batch.circs)
        # values of single-precision states are kept as such
        return values.astype(np.float32) if state["case"]["dtype"] == "c64" else values
    s = state["sv"]
    if kind == "circuit":
        s.reset()
        B.sv_apply_circuit(s.handle, state["circuit"], state["opts"])
        return state["amps"]
    if kind == "step":
        s.reset()
        B.sv_apply_circuit(s.handle, state["circuit"], state["opts"])
        s.swap_bits(0, s.n - 6, 6)
        probs = s.probabilities(state["qubits"])
        return state["amps"], probs.astype(np.float32) if state["case"]["dtype"] == "c64" else probs
    if kind == "gate":
        s.apply_gate(state["u"], state["targets"], state["controls"])
        return state["amps"]
    if kind == "readout":
        return s.readout(state["qubits"], state["terms"], state["uniforms"])
    return s.expect_pauli(state["terms"])


def work(case):
    """Bytes that must cross HBM and real operations of one pass: the state written once where a circuit starts from
    |0...0>, read and written once by a gate (the amplitudes its controls select), read once by read-outs; a
    one-target gate costs 14 operations per amplitude, a dense k-target one 8 * 2^k - 2, a diagonal factor 6."""
    kind = case["kind"]
    if kind == "batch":
        q = range(case["qmin"], case["qmax"] + 1)
        amps = case["count"] * sum(1 << x for x in q) / len(q)
        # 14 for RZ RY as one gate per qubit and layer; the CNOT ladder moves amplitudes; the states stay on chip
        return {"bytes": 8.0 * case["count"] * 2 * case["qmax"],
                "flops": amps * (14.0 * case["layers"] * (case["qmin"] + case["qmax"]) / 2 + 3)}
    n, amp = case["n"], AMP[case["dtype"]]
    size = float(1 << n)
    if kind in ("circuit", "step"):
        ops = 0.0
        for g in _circuit(case["family"], n, case["layers"], np.random.default_rng(0)):
            part = size / (1 << len(g.controls))
            if g.name == "matrix":
                ops += part * (8 * len(g.matrix) - 2)
            elif g.name in ("p", "rz"):
                ops += part * 6 / (2 if g.name == "p" else 1)
            elif g.name not in ("x", "z"):
                ops += part * 14
        bytes_ = size * amp if kind == "circuit" else size * amp * 4
        return {"bytes": bytes_, "flops": ops + (size * 4 if kind == "step" else 0)}
    if kind == "gate":
        part = size / (1 << case["controls"])
        return {"bytes": 2 * part * amp, "flops": part * (8 * (1 << case["targets"]) - 2)}
    if kind == "readout":
        return {"bytes": size * amp, "flops": size * (4 + case["terms"])}
    return {"bytes": size * amp, "flops": size * (4 + 2 * n + 4 * n)}


# --- the same in 64 bits, plain torch -------------------------------------

_H = 1 / math.sqrt(2)


def _u2(name, p):
    if name == "h":
        return [[_H, _H], [_H, -_H]]
    if name == "x":
        return [[0, 1], [1, 0]]
    if name == "z":
        return [[1, 0], [0, -1]]
    if name == "p":
        return [[1, 0], [0, complex(math.cos(p[0]), math.sin(p[0]))]]
    c, s = math.cos(p[0] / 2), math.sin(p[0] / 2)
    if name == "rx":
        return [[c, -1j * s], [-1j * s, c]]
    if name == "ry":
        return [[c, -s], [s, c]]
    if name == "rz":
        return [[complex(c, -s), 0], [0, complex(c, s)]]
    f, l = p[1], p[2]  # u3
    e = lambda x: complex(math.cos(x), math.sin(x))  # noqa: E731
    return [[c, -e(l) * s], [e(f) * s, e(f + l) * c]]


def _apply(psi, n, u, targets, controls):
    """psi <- the gate applied, in place (qubit q is bit q of the index)."""
    qs = sorted(list(targets) + list(controls), reverse=True)
    shape, last = [], n
    for q in qs:
        shape += [1 << (last - 1 - q), 2]
        last = q
    v = psi.view(shape + [1 << last])
    axis = {q: 2 * i + 1 for i, q in enumerate(qs)}

    def part(row):
        index = [slice(None)] * v.dim()
        for c in controls:
            index[axis[c]] = 1
        for b, t in enumerate(targets):
            index[axis[t]] = (row >> b) & 1
        return v[tuple(index)]

    d = 1 << len(targets)
    old = [part(c).clone() for c in range(d)]
    for r in range(d):
        row = [complex(x) for x in u[r]]
        used = [c for c in range(d) if row[c] != 0]
        if used == [r] and row[r] == 1:
            continue
        new = old[used[0]] * row[used[0]]
        for c in used[1:]:
            new.add_(old[c], alpha=row[c])
        part(r).copy_(new)


def _run_exact(gates, n):
    psi = torch.zeros(1 << n, dtype=torch.complex128, device="cuda")
    psi[0] = 1
    for g in gates:
        _apply(psi, n, g.matrix if g.name == "matrix" else _u2(g.name, g.params), g.targets, g.controls)
    return psi


def _sign(n, mask, device):
    """(-1)^popcount(i & mask) for i < 2^n."""
    s = torch.ones(1, dtype=torch.float64, device=device)
    for q in range(n):
        s = torch.cat([s, -s if (mask >> q) & 1 else s])
    return s


def _z_value(prob, n, mask):
    """sum_i p_i (-1)^popcount(i & mask), summing the other qubits out first."""
    qs = [q for q in range(n) if (mask >> q) & 1]
    m = _marginal_exact(prob, n, qs)
    return float((m * _sign(len(qs), (1 << len(qs)) - 1, m.device)).sum())


def _marginal_exact(prob, n, qubits):
    """Distribution over the qubits, bit b of the index = qubits[b]."""
    kept = sorted(qubits)
    shape, last = [], n
    for q in reversed(kept):
        shape += [1 << (last - 1 - q), 2]
        last = q
    v = prob.view(shape + [1 << last])
    v = v.sum(dim=[i for i in range(v.dim()) if i % 2 == 0]) if v.dim() > 1 else v.sum()
    # axes: kept qubits from the highest down; bring them to the order asked for
    order = [len(kept) - 1 - kept.index(q) for q in reversed(list(qubits))]
    return v.permute(order).reshape(-1) if len(kept) > 1 else v.reshape(-1)


def _masks(terms):
    return [sum(1 << q for q, c in enumerate(t) if c == "Z") for t in terms]


def exact(case, seed):
    kind, d = case["kind"], _inputs(case, seed)
    if kind == "batch":
        out = []
        for q, gates, masks in zip(d["qs"], d["gates"], d["masks"]):
            prob = torch.view_as_real(_run_exact(gates, q)).square().sum(-1)
            marg = [_z_value(prob, q, m) for m in masks]
            out += marg
        return np.array(out)
    n = case["n"]
    if kind in ("circuit", "step"):
        psi = _run_exact(d["gates"], n)
        if kind == "circuit":
            return psi
        prob = torch.view_as_real(psi).square().sum(-1)
        probs = _marginal_exact(prob, n, d["qubits"]).cpu().numpy()
        # index bits 0..5 and n-6..n-1 change places in memory
        return psi.view(64, -1, 64).permute(2, 1, 0).reshape(-1), probs
    psi = _random_state(n, case["dtype"], seed).to(torch.complex128)
    if kind == "gate":
        _apply(psi, n, d["u"], d["targets"], d["controls"])
        return psi
    prob = torch.view_as_real(psi).square().sum(-1)
    if kind == "readout":
        return (_marginal_exact(prob, n, d["qubits"]).cpu().numpy(),
                np.array([_z_value(prob, n, m) for m in _masks(d["terms"])]), None)
    out = []
    for t in d["terms"]:
        if "X" in t:
            v = psi.view(-1, 2, 1 << t.index("X"))
            out.append(2 * float((v[:, 0].conj() * v[:, 1]).real.sum()))
        else:
            out.append(_z_value(prob, n, _masks([t])[0]))
    return np.array(out)
