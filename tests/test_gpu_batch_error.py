"""Rounding error of circuits run in register runs (tiles of 2^13 amplitudes)
against sweeps, one gate step at a time in circuit order (tiles of 2^10), over
the expectation values of complex64 ansatz circuits.  The steps are the same and
so is their arithmetic; where the state still has few nonzero amplitudes the
order in which runs take them decides how far one rounding spreads.  Ratio of the
errors over 288 circuits: standard error 2 %, bound 1.04."""
import numpy as np
import pytest

import workloads as W

from paper_2511_14664_amd import _binding as B
from test_gpu_batch import reference

pytestmark = pytest.mark.gpu


def test_error_of_runs_is_that_of_sweeps():
    err = {13: [], 10: []}
    for seed in range(24):
        rng = np.random.default_rng(seed)
        qs = [14 + i % 3 for i in range(12)]
        circs = [W.hea_circuit(q, 4, rng.uniform(0, 2 * np.pi, (4, q)), rng.uniform(0, 2 * np.pi, (4, q))) for q in qs]
        masks = [[1 << i for i in range(q)] + [3 << i for i in range(q - 1)] for q in qs]
        want = reference(circs, qs, masks)
        bt = B.Batch(circs, qs, masks)
        h = B.sv_batch_create(B.SV_C64, bt)
        try:
            for tile, low in ((13, 2), (10, 3)):
                B.sv_batch_set_config(h, tile, low, 2)
                err[tile].append(np.sqrt(np.mean((B.sv_batch_run(h, bt) - want) ** 2)))
        finally:
            B.sv_batch_destroy(h)
    runs, sweeps = float(np.mean(err[13])), float(np.mean(err[10]))
    print(f"runs {runs:.3e} sweeps {sweeps:.3e} ratio {runs / sweeps:.3f}", flush=True)
    assert runs <= 1.04 * sweeps
