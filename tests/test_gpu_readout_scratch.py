"""Scratch of a fused read-out: partial sums only of the strings that it has.
Eighteen bins above bit 11 of a 30-qubit state leave one 4096-amplitude segment
per workgroup, 2^18 of them: 2 MiB each of folded sums, block totals and results,
and 2 MiB per string (32 of them: 64 MiB)."""
import numpy as np
import pytest
import torch

from paper_2511_14664_amd import _binding as B

pytestmark = pytest.mark.gpu


def test_scratch_without_strings():
    n, mib = 30, 1 << 20
    h = B.sv_create(n, B.SV_C64)
    try:
        B.sv_reset(h)
        B.sv_synchronize(h)
        free = torch.cuda.mem_get_info()[0]
        u = np.random.default_rng(1).random(10)
        probs, _, shots = B.sv_readout(h, list(range(12, n)), [], u)
        took = free - torch.cuda.mem_get_info()[0]
        print(f"{took / mib:.1f} MiB", flush=True)
        assert probs[0] == 1.0 and not np.any(shots)
        assert took <= 16 * mib
        z = ["Z" + "I" * (n - 1), "I" * (n - 1) + "Z"]
        probs, values, shots = B.sv_readout(h, list(range(12, n)), z, u)
        assert probs[0] == 1.0 and np.array_equal(values, [1.0, 1.0]) and not np.any(shots)
    finally:
        B.sv_destroy(h)
