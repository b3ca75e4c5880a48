"""Circuits of a batch whose gates run in register runs (tiles of 2^11 to 2^13
amplitudes): every step type on random qubits in both orders, so that runs cut
and reorder them in every way, and Z strings over bits inside and outside the
tile, up to 64 of them.  Against the FP64 reference, bounds as in test_gpu_batch:
FP64 rounding (1e-12), or FP32 rounding of a few hundred gates (2e-5)."""
import numpy as np
import pytest

from workloads import Gate

from paper_2511_14664_amd import _binding as B
from test_gpu_batch import ETOL, reference, say

pytestmark = pytest.mark.gpu


def unitary(rng, d):
    q, r = np.linalg.qr(rng.normal(size=(d, d)) + 1j * rng.normal(size=(d, d)))
    return q * (np.diag(r) / np.abs(np.diag(r)))


def mixed_circuit(q, count, rng):
    out = []
    for _ in range(count):
        a, b = (int(x) for x in rng.choice(q, 2, replace=False))
        kind = int(rng.integers(5))
        if kind == 0:
            out.append(Gate("matrix", (a,), (), (), unitary(rng, 2)))
        elif kind == 1:
            out.append(Gate("ry", (a,), (), (float(rng.uniform(0, 6)),)))
        elif kind == 2:
            out.append(Gate("x", (a,), (b,)))
        elif kind == 3:
            out.append(Gate("rz", (a,), (b,), (float(rng.uniform(0, 6)),)))
        else:
            out.append(Gate("matrix", (a, b), (), (), unitary(rng, 4)))
    return out


@pytest.mark.parametrize("dtype", [B.SV_C128, B.SV_C64], ids=["c128", "c64"])
@pytest.mark.parametrize("tile,low,fuse", [(11, 2, 1), (11, 0, 2), (12, 1, 2), (12, 3, 1), (13, 2, 2), (13, 0, 1)])
def test_runs_match_reference(dtype, tile, low, fuse):
    if dtype == B.SV_C128 and tile == 13:
        pytest.skip("complex128 tiles end at 2^12")
    rng = np.random.default_rng(100 * tile + 10 * low + fuse)
    qs = [tile - 1, tile, tile + 1, tile + 3]
    circs = [mixed_circuit(q, 60 + 5 * q, rng) for q in qs] + [[]]
    qs = qs + [tile + 1]
    masks = [[int(m) for m in rng.integers(0, 1 << q, count)] for q, count in zip(qs, [5, 64, 17, 64, 3])]
    want = reference(circs, qs, masks)
    bt = B.Batch(circs, qs, masks)
    h = B.sv_batch_create(dtype, bt)
    try:
        B.sv_batch_set_config(h, tile, low, fuse)
        say(f"tile {tile} low {low} fuse {fuse}")
        for _ in range(3):  # replays of one graph
            got = B.sv_batch_run(h, bt)
            assert float(np.max(np.abs(got - want))) <= ETOL[dtype]
    finally:
        B.sv_batch_destroy(h)
