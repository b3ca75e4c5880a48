"""Threads that run circuits of small states side by side, each with a handle and
a stream of its own and programs of different LDS sizes (a state of 64 KiB with
one table of steps, with matrices of six targets, and a state of a few bytes):
every result against the FP64 reference, 2e-5 (complex64) and 1e-12 (complex128)
as for one caller."""
import threading

import numpy as np
import pytest
import torch

import oracle
import workloads as W
from workloads import Gate

import paper_2511_14664_amd as svm
from paper_2511_14664_amd import _binding as B

pytestmark = pytest.mark.gpu


def test_programs_of_different_sizes_in_threads():
    rng = np.random.default_rng(2)
    wide = [Gate("matrix", tuple(int(q) for q in rng.choice(12, 6, replace=False)), (), (), W.haar_unitary(rng, 64))
            for _ in range(5)]
    work = [(13, B.SV_C64, W.layered_u3_pairing(13, 2, 1, "cx")), (12, B.SV_C128, wide),
            (12, B.SV_C128, W.layered_u3_pairing(12, 12, 2, "cx_or_cz")), (4, B.SV_C64, W.layered_u3_pairing(4, 3, 3, "cx"))]
    wants = [oracle.run(g, n) for n, _, g in work]
    errs = [None] * len(work)
    start = threading.Barrier(len(work))

    def run(i):
        n, dtype, gates = work[i]
        with svm.StateVector(n, dtype, stream=torch.cuda.Stream()) as s:
            circ = B.Circuit(gates)
            start.wait()
            worst = 0.0
            for _ in range(40):
                s.reset()
                s.apply_circuit(circ)
                worst = max(worst, float(np.max(np.abs(s.to_host() - wants[i]))))
            errs[i] = worst

    threads = [threading.Thread(target=run, args=(i,)) for i in range(len(work))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for (n, dtype, _), e in zip(work, errs):
        assert e is not None and e <= (2e-5 if dtype == B.SV_C64 else 1e-12), (n, dtype, errs)
