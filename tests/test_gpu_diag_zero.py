"""Diagonal steps of a pass whose phase angles are zero, in all of its passes or
in some: the step has no terms and leaves the amplitudes alone, whatever an
earlier launch left in LDS.  Against the FP64 reference.  Bound: FP32 rounding
of amplitudes below 2^-5 over a few hundred gates, 2e-6; FP64 1e-13."""
import numpy as np
import pytest

import oracle
import workloads as W
from workloads import Gate

from paper_2511_14664_amd import _binding as B

pytestmark = pytest.mark.gpu


def layers(n, angle):
    """H, then twice: every controlled phase (angle(layer) each), RX on every qubit."""
    g = [Gate("h", (q,)) for q in range(n)]
    for k in range(2):
        g += [Gate("p", (b,), (a,), (angle(k),)) for a in range(n) for b in range(a)]
        g += [Gate("rx", (q,), (), (0.3 + 0.1 * q,)) for q in range(n)]
    return g


ANGLES = {"all": lambda k: 0.0, "first": lambda k: 0.0 if k == 0 else 0.37, "last": lambda k: 0.37 if k == 0 else 0.0}


@pytest.mark.parametrize("dtype,prec", [(B.SV_C128, B.SV_PREC_NATIVE), (B.SV_C64, B.SV_PREC_NATIVE),
                                        (B.SV_C64, B.SV_PREC_BF16X6)], ids=["c128", "c64", "c64-split"])
@pytest.mark.parametrize("n", [14, 17])
@pytest.mark.parametrize("zero", list(ANGLES))
def test_zero_angles(zero, n, dtype, prec):
    opts = B.make_opts(B.SV_PLAN_PASSES, 4, prec)
    gates = layers(n, ANGLES[zero])
    h = B.sv_create(n, dtype)
    try:
        # angles of every diagonal step, left behind in LDS
        B.sv_copy_from_host(h, dtype, W.random_state(n, 1))
        B.sv_apply_circuit(h, layers(n, lambda k: 1.1 + k), opts)
        B.sv_copy_from_host(h, dtype, W.random_state(n, n))
        start = B.sv_copy_to_host(h, n, dtype).astype(np.complex128)
        B.sv_apply_circuit(h, gates, opts)
        got = B.sv_copy_to_host(h, n, dtype)
        want = oracle.run(gates, n, start)
        assert np.max(np.abs(got - want)) <= (1e-13 if dtype == B.SV_C128 else 2e-6)
    finally:
        B.sv_destroy(h)
