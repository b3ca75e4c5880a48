"""Expectation values that share reads of the state: every string of a small
state in one launch, many Z strings by a Walsh transform, strings whose X and
Y positions fit one tile together, against the FP64 oracle on the state the
GPU holds.  All sums are FP64 over at most 2^22 products of a normalised
state, so their rounding stays below 22 * 2^-53 * 2 < 1e-14 per unit of the
sum of moduli (at most 1); the bound used is 1e-12, as for the other
read-outs."""
import numpy as np
import pytest

import oracle
import workloads as W

from paper_2511_14664_amd import _binding as B

pytestmark = pytest.mark.gpu


def string(n, at):
    return "".join(at.get(q, "I") for q in range(n))


def terms_for(n, seed):
    """One-site X and Y on every qubit, neighbour XX, YY, XY, XYZ, Z strings
    (more than one batch), long X strings that fit no tile, random strings."""
    rng = np.random.default_rng(seed)
    t = [string(n, {q: p}) for p in "XYZ" for q in range(n)]
    for a, b in (("X", "X"), ("Y", "Y"), ("X", "Y")):
        t += [string(n, {q: a, (q + 1) % n: b}) for q in range(n)] if n > 1 else []
    if n > 2:
        t += [string(n, {q: "X", (q + 1) % n: "Y", (q + 2) % n: "Z"}) for q in range(n)]
    t += ["I" * n, "X" * n, "Y" * n, "Z" * n]
    t += ["".join(rng.choice(list("IZ"), size=n)) for _ in range(130)]
    t += ["".join(rng.choice(list("IXYZ"), size=n)) for _ in range(6)]
    return [t[i] for i in rng.permutation(len(t))]


# 1..19: all strings in one launch (12 / 13: one / two chunks a string);
# 20, 21: fewer tiles than workgroups, and more than one per workgroup
@pytest.mark.parametrize("dtype", [B.SV_C64, B.SV_C128], ids={B.SV_C64: "c64", B.SV_C128: "c128"}.get)
@pytest.mark.parametrize("n", [1, 3, 12, 13, 19, 20, 21])
def test_shared_reads_match_oracle(dtype, n):
    h = B.sv_create(n, dtype)
    try:
        B.sv_copy_from_host(h, dtype, W.random_state(n, 31 + n))
        if n >= 13:
            B.sv_swap_bits(h, 1, n - 4, 3)  # physical positions other than the logical ones
        psi = B.sv_copy_to_host(h, n, dtype).astype(np.complex128)
        terms = terms_for(n, n)
        if n > 18:
            terms = terms[:160]
        for sub in (terms, terms[:3], [t for t in terms if set(t) <= set("IZ")][:33],
                    [t for t in terms if "X" in t or "Y" in t][:17]):
            got = B.sv_expect_pauli(h, sub)
            want = np.array([oracle.expect_pauli(psi, t).real for t in sub])
            assert float(np.max(np.abs(got - want))) <= 1e-12
            if len(sub) <= B.SV_NOALLOC_MAX_TERMS:
                assert np.array_equal(B.sv_expect_pauli_noalloc(h, sub), got)
    finally:
        B.sv_destroy(h)
