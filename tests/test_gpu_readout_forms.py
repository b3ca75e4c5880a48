"""sv_readout and sv_probabilities over every placement of the marginal's
physical bits: inside a segment of 4096 amplitudes (with and without the bits a
thread's loads differ in), around its edge (11, 12, 13), in the gaps of the bits
that a workgroup sums over, and only above; and shots from states that are
mostly zero.  Bounds as in test_gpu_readout: sums of FP64 squares of one state
in another order, 1e-13 between the two routes and 1e-12 against the FP64
reference.
"""
import numpy as np
import pytest

import workloads as W

from paper_2511_14664_amd import _binding as B
from test_gpu_readout import check, say, z_terms

pytestmark = pytest.mark.gpu

DTYPES = [B.SV_C128, B.SV_C64]
DNAME = {B.SV_C128: "c128", B.SV_C64: "c64"}


@pytest.mark.parametrize("dtype", DTYPES, ids=DNAME.get)
@pytest.mark.parametrize("n,bins", [
    (14, [12]), (14, [13, 12]), (14, [11, 12, 0]), (14, [8, 9, 10, 11]), (14, [13, 7]),
    (18, [12, 14, 16]), (18, [13, 15, 17]), (18, [17, 8, 12]), (18, list(range(8, 18))),
    (20, [19, 18, 17, 16, 15]), (20, [12, 13, 9]), (20, list(range(9, -1, -1))), (20, list(range(12))),
])
def test_marginal_bits(dtype, n, bins):
    h = B.sv_create(n, dtype)
    try:
        B.sv_copy_from_host(h, dtype, W.random_state(n, 7 * n + len(bins)))
        u = W.uniforms(n, 300)
        say(f"n={n} {DNAME[dtype]} bins {bins}")
        check(h, n, dtype, bins, z_terms(n, 9, n), u)
        check(h, n, dtype, bins, [], u)
        check(h, n, dtype, bins, z_terms(n, 33, n) + ["X" + "Z" * (n - 2) + "Y"], u)
    finally:
        B.sv_destroy(h)


@pytest.mark.parametrize("dtype", DTYPES, ids=DNAME.get)
def test_grid_limit(dtype):
    """More segments than one workgroup each: n = 26 leaves two bits to sum
    over, contiguous or split by bins (bits 12 and 14)."""
    n = 26
    h = B.sv_create(n, dtype)
    try:
        B.sv_reset(h)
        for q in range(n):
            c, s = np.cos(0.2 + 0.05 * q), np.sin(0.2 + 0.05 * q)
            B.sv_apply_gate(h, np.array([[c, -s], [s, c]], dtype=np.complex128), [q])
        p1 = np.sin(0.2 + 0.05 * np.arange(n)) ** 2
        qmap = [int(x) for x in B.sv_qubit_map(h, n)]
        tol = 1e-12 if dtype == B.SV_C128 else 26 * 2e-6  # a gate's rounding times 26 gates
        for phys in ([25, 24, 23], [12, 14], [13, 3], [12, 10]):
            bins = [qmap.index(p) for p in phys]
            terms = ["I" * q + "Z" + "I" * (n - 1 - q) for q in (0, 12, 13, 25)]
            say(f"{DNAME[dtype]} physical bins {phys}")
            probs, ex, shots = B.sv_readout(h, bins, terms, W.uniforms(3, 100))
            want = np.array([np.prod([p1[q] if (x >> b) & 1 else 1 - p1[q] for b, q in enumerate(bins)])
                             for x in range(1 << len(bins))])
            assert np.max(np.abs(probs - want)) <= tol
            assert np.max(np.abs(np.sort(ex) - np.sort([1 - 2 * p1[q] for q in (0, 12, 13, 25)]))) <= 2 * tol
            assert np.max(np.abs(probs - B.sv_probabilities(h, bins))) <= 1e-13
            assert np.mean(shots == B.sv_sample(h, W.uniforms(3, 100))) >= 0.99
    finally:
        B.sv_destroy(h)


@pytest.mark.parametrize("dtype", DTYPES, ids=DNAME.get)
@pytest.mark.parametrize("n", [9, 11, 14, 17])
def test_shots_of_sparse_states(dtype, n):
    """Uniforms at both ends of [0, 1) and between them only ever give indices
    of nonzero amplitudes, the first and the last one at the ends."""
    N = 1 << n
    rng = np.random.default_rng(n)
    for nz in ([0], [N - 1], [N // 2 - 1, N // 2], sorted(rng.choice(N, 40, replace=False).tolist())):
        psi = np.zeros(N, dtype=np.complex128)
        psi[nz] = 1 / np.sqrt(len(nz))
        u = np.concatenate([[0.0, np.nextafter(1.0, 0.0)], np.arange(len(nz)) / len(nz), rng.random(200)])
        h = B.sv_create(n, dtype)
        try:
            B.sv_copy_from_host(h, dtype, psi)
            say(f"n={n} {DNAME[dtype]} {len(nz)} nonzero amplitudes")
            got = B.sv_sample(h, u)
            fused = B.sv_readout(h, None, [], u)[2]
            for s in (got, fused):
                assert set(int(x) for x in s) <= set(nz)
                assert int(s[0]) == nz[0] and int(s[1]) == nz[-1]
        finally:
            B.sv_destroy(h)
