"""The number of Z strings up to which the sweep that adds each string up is
taken (8; 16 on complex64 states of at least 25 qubits), on both sides of each
line, against FP64 sums on the GPU.  All sums are FP64 over 2^25 products of a
normalised state: their rounding stays below 25 * 2^-53 * 2 < 1e-14 per unit
of the sum of moduli (at most 1); the bound is 1e-12, as for the other
read-outs.  A call must also give the same with its strings in two halves."""
import numpy as np
import pytest

import workloads as W

from paper_2511_14664_amd import _binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nz", [1, 8, 9, 15, 16, 17])
@pytest.mark.parametrize("n,dtype", [(20, B.SV_C64), (24, B.SV_C64), (25, B.SV_C64), (25, B.SV_C128)],
                         ids=["20q-c64", "24q-c64", "25q-c64", "25q-c128"])
def test_z_strings_on_both_sides_of_the_line(n, dtype, nz):
    import torch

    dev = torch.device("cuda", 0)
    ct = torch.complex64 if dtype == B.SV_C64 else torch.complex128
    a = torch.empty(1 << n, dtype=ct, device=dev)
    rng = np.random.default_rng(n + nz)
    terms = ["".join(rng.choice(list("IZ"), size=n)) for _ in range(nz)]
    h = B.sv_create_on(a.data_ptr(), a.numel() * a.element_size(), n, dtype, 0)
    try:
        a.copy_(torch.randn(1 << n, dtype=ct, device=dev, generator=torch.Generator(dev).manual_seed(n)))
        a /= torch.linalg.vector_norm(a)
        torch.cuda.synchronize()
        got = B.sv_expect_pauli(h, terms)
        halves = np.concatenate([B.sv_expect_pauli(h, terms[:nz // 2]), B.sv_expect_pauli(h, terms[nz // 2:])])
        noalloc = B.sv_expect_pauli_noalloc(h, terms)
    finally:
        B.sv_destroy(h)
    p = a.real.double() ** 2 + a.imag.double() ** 2
    for t, g in zip(terms, got):
        q = p
        for k in range(n):  # fold index bit k away: x0 + x1 or x0 - x1
            v = q.view(-1, 2)
            q = v[:, 0] - v[:, 1] if t[k] == "Z" else v[:, 0] + v[:, 1]
        assert abs(float(q[0]) - g) <= 1e-12, t
    assert float(np.max(np.abs(got - halves))) <= 1e-12
    assert np.array_equal(noalloc, got)
