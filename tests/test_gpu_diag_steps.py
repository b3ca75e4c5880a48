"""Runs of phase gates inside a pass, done as one diagonal step: controlled
phases, ZZ rotations, phases with one or two qubits outside the tile and phases
of three and four qubits (which stay blocks), between gates that they cannot
pass.  Against the FP64 reference; bound: FP32 rounding of the amplitudes (which
are below 2^-5) over a few hundred gates, 2e-6, FP64 1e-13.
"""
import numpy as np
import pytest

import oracle
import workloads as W
from workloads import Gate

from paper_2511_14664_amd import _binding as B

pytestmark = pytest.mark.gpu


def qft(n):
    g = []
    for q in range(n):
        g.append(Gate("h", (q,)))
        g += [Gate("p", (j,), (q,), (np.pi / 2 ** (j - q),)) for j in range(q + 1, n)]
    return g


def zz_layers(n, layers, rng):
    g = []
    for _ in range(layers):
        for a in range(n):
            for b in (int(x) for x in rng.choice(n, 3, replace=False)):
                if a != b:
                    g += [Gate("x", (b,), (a,)), Gate("rz", (b,), (), (float(rng.uniform(0, 6)),)), Gate("x", (b,), (a,))]
        g += [Gate("rx", (q,), (), (float(rng.uniform(0, 3)),)) for q in range(0, n, 2)]
    return g


def phases(n, count, rng):
    g = []
    for k in range(count):
        m = int(rng.choice([1, 2, 2, 2, 2, 2, 3, 4]))
        qs = [int(x) for x in rng.choice(n, m, replace=False)]
        g.append(Gate("p", (qs[0],), tuple(qs[1:]), (float(rng.uniform(0, 6)),)))
        if k % 40 == 39:
            g.append(Gate("h", (int(rng.integers(n)),)))
        if k % 60 == 59:
            a, b = (int(x) for x in rng.choice(n, 2, replace=False))
            g.append(Gate("x", (a,), (b,)))
    return g


CIRCUITS = {
    "qft": lambda n, rng: qft(n),
    "zz": lambda n, rng: zz_layers(n, 3, rng),
    "phases": lambda n, rng: [Gate("h", (q,)) for q in range(n)] + phases(n, 300, rng),
}


@pytest.mark.parametrize("dtype,prec", [(B.SV_C128, B.SV_PREC_NATIVE), (B.SV_C64, B.SV_PREC_NATIVE),
                                        (B.SV_C64, B.SV_PREC_BF16X6)], ids=["c128", "c64", "c64-split"])
@pytest.mark.parametrize("n", [13, 16, 19])
@pytest.mark.parametrize("name", list(CIRCUITS))
def test_diagonal_steps(name, n, dtype, prec):
    gates = CIRCUITS[name](n, np.random.default_rng(n))
    h = B.sv_create(n, dtype)
    try:
        for tile in (0, 13) if dtype == B.SV_C64 and prec == B.SV_PREC_NATIVE and n > 13 else (0,):
            B.sv_copy_from_host(h, dtype, W.random_state(n, n))
            start = B.sv_copy_to_host(h, n, dtype).astype(np.complex128)
            st = B.sv_apply_circuit(h, gates, B.make_opts(B.SV_PLAN_PASSES, 4, prec, 0, 0, tile))
            print(f"{name} n={n} tile {tile}: {len(gates)} gates, {st['sweeps']} sweeps", flush=True)
            got = B.sv_copy_to_host(h, n, dtype)
            want = oracle.run(gates, n, start)
            assert np.max(np.abs(got - want)) <= (1e-13 if dtype == B.SV_C128 else 2e-6)
    finally:
        B.sv_destroy(h)
