"""Angles of phase gates in complex64 passes are rounded, not cut, to 2^-32 turns.
Controlled phases of (k + 0.9) / 2^32 turns on |1..1>, whose amplitude collects
every one of them: cut, each falls short by 0.9 of 2^-32 turns, rounded each is
0.1 off.  Bound on the phase: 0.1 * 2^-32 turns a gate, and per layer of gates
the rounding of a sine and cosine and of one complex product, 3 * 2^-24."""
import math

import numpy as np
import pytest

from workloads import Gate

from paper_2511_14664_amd import _binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [B.SV_PREC_NATIVE, B.SV_PREC_BF16X6], ids=["native", "split"])
@pytest.mark.parametrize("n", [16, 24])
def test_angles_are_rounded(n, prec):
    rng = np.random.default_rng(n)
    layers, count, turns = 8, 0, 0
    gates = [Gate("x", (q,)) for q in range(n)]
    for _ in range(layers):
        for a in range(n):
            for b in range(a):
                k = 10 * int(rng.integers(1 << 32)) + 9  # tenths of 2^-32 turns
                turns += k
                count += 1
                gates.append(Gate("p", (b,), (a,), (2 * math.pi * k / (10 * 2 ** 32),)))
        # the identity, which the phases of two layers cannot pass
        gates += [Gate("x", (q,)) for q in range(n) for _ in range(2)]
    want = 2 * math.pi * (turns % (10 * 2 ** 32)) / (10 * 2 ** 32)
    h = B.sv_create(n, B.SV_C64)
    try:
        B.sv_reset(h)
        B.sv_apply_circuit(h, gates, B.make_opts(B.SV_PLAN_PASSES, 5, prec))
        got = complex(B.sv_copy_to_host(h, n, B.SV_C64, (1 << n) - 1, 1)[0])
    finally:
        B.sv_destroy(h)
    off = abs(math.remainder(math.atan2(got.imag, got.real) - want, 2 * math.pi))
    bound = count * 0.1 * 2.0 ** -32 * 2 * math.pi + layers * 3 * 2.0 ** -24
    print(f"n={n}: {count} gates, phase off by {off:.3g}, bound {bound:.3g}", flush=True)
    assert off <= bound
