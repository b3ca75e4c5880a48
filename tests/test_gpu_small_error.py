"""Rounding error of fused blocks on states that fit LDS against that of one
launch per block (taken while sweeps are timed), both measured in extended
precision.  Both form a block's complex products alike, so the errors are equal
but for the order of the sums; three real products per complex one where the
launches take four would make them 1.4 times as large.  The errors of 60 blocks
are independent vectors of at least 2^9 components: their norms agree to about
1 %, the bound is 1.15."""
import numpy as np
import pytest

import workloads as W
from workloads import Gate

from paper_2511_14664_amd import _binding as B

pytestmark = pytest.mark.gpu


def apply_long(psi, n, u, targets):
    k = len(targets)
    v = psi.reshape((2,) * n)
    # axis of qubit q is n - 1 - q; matrix index bit b is targets[b]
    src = [n - 1 - t for t in reversed(targets)]
    v = np.moveaxis(v, src, range(k))
    shape = v.shape
    v = (u @ v.reshape(1 << k, -1)).reshape(shape)
    return np.ascontiguousarray(np.moveaxis(v, range(k), src)).reshape(-1)


@pytest.mark.parametrize("dtype", [B.SV_C64, B.SV_C128], ids=["c64", "c128"])
@pytest.mark.parametrize("n", [8, 9, 10, 11, 12])
@pytest.mark.parametrize("k", [3, 4, 5, 6])
def test_error_of_a_block_is_that_of_a_launch(k, n, dtype):
    rng = np.random.default_rng(100 * k + n)
    cast = np.complex64 if dtype == B.SV_C64 else np.complex128
    # matrices that the state's precision holds as they are
    gates = [Gate("matrix", tuple(int(q) for q in rng.choice(n, k, replace=False)), (), (),
                  W.haar_unitary(rng, 1 << k).astype(cast).astype(np.complex128)) for _ in range(60)]
    start = W.random_state(n, n).astype(cast)
    want = start.astype(np.clongdouble)
    for g in gates:
        want = apply_long(want, n, g.matrix.astype(np.clongdouble), g.targets)
    h = B.sv_create(n, dtype)
    err = {}
    try:
        for timed in (True, False):
            B.sv_copy_from_host(h, dtype, start)
            B.sv_profile_enable(h, timed)
            B.sv_apply_circuit(h, gates, B.make_opts(B.SV_PLAN_PLAIN))
            B.sv_profile_enable(h, False)
            assert len(B.sv_profile_read(h)) == (len(gates) if timed else 0)
            d = B.sv_copy_to_host(h, n, dtype).astype(np.clongdouble) - want
            err[timed] = float(np.sqrt(np.sum(d.real ** 2 + d.imag ** 2)))
    finally:
        B.sv_destroy(h)
    print(f"k={k} n={n}: step {err[False]:.3e} launch {err[True]:.3e} ratio {err[False] / err[True]:.3f}", flush=True)
    assert err[False] <= 1.15 * err[True]
