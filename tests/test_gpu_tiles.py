"""Tile kernels at the edges of their addressing: gates of two to six targets
with up to eight controls (a tile's bits and the controls outside it), and pass
blocks on every kind of tile slots (low and high bits that share LDS banks, the
pass kernels' lane layouts), against the FP64 reference.  Bounds: a gate of 2^k
products per amplitude in FP64 (1e-13) or FP32 (2^k half ulps, 64 * 2^-24), and
as many times that as there are gates.
"""
import numpy as np
import pytest

import oracle
import workloads as W
from workloads import Gate

from paper_2511_14664_amd import _binding as B

pytestmark = pytest.mark.gpu

TOL = {B.SV_C128: 1e-13, B.SV_C64: 64 * 2.0 ** -24}
DNAME = {B.SV_C128: "c128", B.SV_C64: "c64"}


def unitary(rng, d):
    q, r = np.linalg.qr(rng.normal(size=(d, d)) + 1j * rng.normal(size=(d, d)))
    return q * (np.diag(r) / np.abs(np.diag(r)))


@pytest.mark.parametrize("dtype", [B.SV_C128, B.SV_C64], ids=DNAME.get)
@pytest.mark.parametrize("k", [2, 3, 4, 5, 6])
@pytest.mark.parametrize("c", [0, 2, 3, 5, 8])
def test_targets_and_controls(dtype, k, c):
    n = max(16, 13 + c)
    rng = np.random.default_rng(100 * k + c)
    psi = W.random_state(n, k + c)
    h = B.sv_create(n, dtype)
    try:
        for _ in range(2):
            B.sv_copy_from_host(h, dtype, psi)
            host = B.sv_copy_to_host(h, n, dtype).astype(np.complex128)
            qs = [int(x) for x in rng.choice(n, k + c, replace=False)]
            U = unitary(rng, 1 << k)
            print(f"n={n} {DNAME[dtype]} targets {qs[:k]} controls {qs[k:]}", flush=True)
            B.sv_apply_gate(h, U, qs[:k], qs[k:])
            got = B.sv_copy_to_host(h, n, dtype)
            want = oracle.apply_matrix(host, U, qs[:k], qs[k:])
            assert np.max(np.abs(got - want)) <= TOL[dtype]
    finally:
        B.sv_destroy(h)


@pytest.mark.parametrize("dtype,prec", [(B.SV_C128, B.SV_PREC_NATIVE), (B.SV_C64, B.SV_PREC_NATIVE),
                                        (B.SV_C64, B.SV_PREC_BF16X6)], ids=["c128", "c64", "c64-split"])
@pytest.mark.parametrize("qubits", [[0, 4, 8, 11], [0, 1, 5, 9], [0, 2, 6, 10], [0, 3, 7, 11], [4, 8, 12, 3],
                                    [11, 10, 9, 8], [3, 2, 1, 0], [13, 5, 1, 9], [12, 13, 0, 6]])
def test_pass_blocks_on_slots(dtype, prec, qubits):
    n = 19
    rng = np.random.default_rng(sum(qubits))
    other = [q for q in range(n) if q not in qubits]
    # two blocks on the slots under test, others around them on overlapping ones
    gates = [Gate("matrix", tuple(qubits), (), (), unitary(rng, 16)),
             Gate("matrix", tuple([qubits[0], qubits[2], other[0], other[1]]), (), (), unitary(rng, 16)),
             Gate("matrix", tuple(qubits[::-1]), (), (), unitary(rng, 16)),
             Gate("p", (qubits[1],), (other[-1],), (0.7,)),
             Gate("matrix", tuple([other[0], qubits[3], other[1], qubits[1]]), (), (), unitary(rng, 16))]
    h = B.sv_create(n, dtype)
    try:
        psi = W.random_state(n, 5)
        for tile in (0, 13 if dtype == B.SV_C64 and prec == B.SV_PREC_NATIVE else 12):
            B.sv_copy_from_host(h, dtype, psi)
            host = B.sv_copy_to_host(h, n, dtype).astype(np.complex128)
            st = B.sv_apply_circuit(h, gates, B.make_opts(B.SV_PLAN_PASSES, 4, prec, 8, 8, tile))
            print(f"{qubits} tile {tile} sweeps {st['sweeps']}", flush=True)
            assert st["sweeps"] < len(gates)
            want = host
            for g in gates:
                want = oracle.apply_gate(want, g)
            got = B.sv_copy_to_host(h, n, dtype)
            assert np.max(np.abs(got - want)) <= len(gates) * TOL[dtype]
    finally:
        B.sv_destroy(h)
