"""Blocks of four to six targets with controls on states that fit LDS: against
the FP64 reference (2e-5 complex64, 1e-12 complex128), with the rounding error of
a launch per block (bound 1.15, as for blocks without controls; the norms of the
errors of 40 blocks, each on a part of the state, agree to a few percent), and no
slower than the launches (taken while sweeps are timed)."""
import time

import numpy as np
import pytest

import oracle
import workloads as W
from workloads import Gate

from paper_2511_14664_amd import _binding as B

pytestmark = pytest.mark.gpu

DTYPES = [B.SV_C64, B.SV_C128]
IDS = {B.SV_C64: "c64", B.SV_C128: "c128"}.get
TOL = {B.SV_C64: 2e-5, B.SV_C128: 1e-12}


def controlled(n, k, c, count, rng, cast):
    gates = []
    for _ in range(count):
        q = [int(x) for x in rng.choice(n, k + c, replace=False)]
        gates.append(Gate("matrix", tuple(q[:k]), tuple(q[k:]), (),
                          W.haar_unitary(rng, 1 << k).astype(cast).astype(np.complex128)))
    return gates


# groups of a step: 2^(n - k - c), from one to the most; 16 and more run on the matrix cores
@pytest.mark.parametrize("dtype", DTYPES, ids=IDS)
@pytest.mark.parametrize("n", [5, 8, 9, 10, 11, 12, 13])
def test_values(n, dtype):
    if n == 13 and dtype == B.SV_C128:
        n = 7  # the largest complex128 state here has 12 qubits
    rng = np.random.default_rng(n)
    cast = np.complex64 if dtype == B.SV_C64 else np.complex128
    h = B.sv_create(n, dtype)
    try:
        for k in range(2, min(6, n) + 1):
            for c in range(1, min(n - k, 8) + 1):
                gates = controlled(n, k, c, 3, rng, cast)
                B.sv_copy_from_host(h, dtype, W.random_state(n, n))
                start = B.sv_copy_to_host(h, n, dtype).astype(np.complex128)
                B.sv_apply_circuit(h, gates, B.make_opts(B.SV_PLAN_PLAIN))
                got = B.sv_copy_to_host(h, n, dtype)
                d = float(np.max(np.abs(got - oracle.run(gates, n, start))))
                assert d <= TOL[dtype], (n, k, c, d)
    finally:
        B.sv_destroy(h)


def apply_long(psi, n, g):
    """One gate in extended precision."""
    k, t = len(g.targets), g.targets
    v = psi.reshape((2,) * n)
    src = [n - 1 - q for q in reversed(t)]
    v = np.moveaxis(v, src, range(k)).copy()
    axes = sorted(n - 1 - q for q in g.controls)
    # the controls' axes after the targets' have moved to the front
    rest = [a for a in range(n) if a not in src]
    sel = (slice(None),) * k + tuple(1 if a in axes else slice(None) for a in rest)
    part = v[sel]
    v[sel] = (g.matrix.astype(np.clongdouble) @ part.reshape(1 << k, -1)).reshape(part.shape)
    return np.ascontiguousarray(np.moveaxis(v, range(k), src)).reshape(-1)


CASES = [(B.SV_C64, 11, 4, 1), (B.SV_C64, 12, 5, 1), (B.SV_C64, 13, 6, 1), (B.SV_C64, 13, 4, 2), (B.SV_C64, 11, 6, 1),
         (B.SV_C128, 11, 4, 1), (B.SV_C128, 12, 6, 1), (B.SV_C128, 12, 4, 2), (B.SV_C128, 12, 5, 2)]


@pytest.mark.parametrize("dtype,n,k,c", CASES, ids=lambda x: str(x))
def test_error_and_time_of_launches(dtype, n, k, c):
    rng = np.random.default_rng(n * 100 + k * 10 + c)
    cast = np.complex64 if dtype == B.SV_C64 else np.complex128
    gates = controlled(n, k, c, 40, rng, cast)
    start = W.random_state(n, n).astype(cast)
    want = start.astype(np.clongdouble)
    for g in gates:
        want = apply_long(want, n, g)
    circ, opts = B.Circuit(gates), B.make_opts(B.SV_PLAN_PLAIN)
    h = B.sv_create(n, dtype)
    err, took = {}, {}
    try:
        for timed in (True, False):
            B.sv_profile_enable(h, timed)
            B.sv_copy_from_host(h, dtype, start)
            B.sv_apply_circuit(h, circ, opts)
            d = B.sv_copy_to_host(h, n, dtype).astype(np.clongdouble) - want
            err[timed] = float(np.sqrt(np.sum(d.real ** 2 + d.imag ** 2)))
            runs = []
            for _ in range(7):
                t = time.perf_counter()
                B.sv_apply_circuit(h, circ, opts)
                B.sv_synchronize(h)
                runs.append(time.perf_counter() - t)
            took[timed] = min(runs)
            B.sv_profile_read(h)
    finally:
        B.sv_destroy(h)
    print(f"n={n} k={k} c={c}: step {err[False]:.3e} {took[False] * 1e6:.0f} us, "
          f"launch {err[True]:.3e} {took[True] * 1e6:.0f} us", flush=True)
    assert err[False] <= 1.15 * err[True]
    assert took[False] <= took[True]
