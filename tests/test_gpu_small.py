"""Circuits on states that fit one workgroup's LDS run as steps of one launch:
every gate shape and state size at its edges, against the FP64 oracle, with
the tolerances of the per-launch sweeps (1e-12 complex128, 2e-5 complex64 at
depth <= 200, tests/test_gpu_parity.py), and against the launch-per-sweep
path (taken while sweeps are timed)."""
import numpy as np
import pytest

import oracle
import workloads as W

from paper_2511_14664_amd import _binding as B

pytestmark = pytest.mark.gpu

DTYPES = [B.SV_C64, B.SV_C128]
IDS = {B.SV_C64: "c64", B.SV_C128: "c128"}.get
TOL = {B.SV_C64: 2e-5, B.SV_C128: 1e-12}


def mixed_gates(n, count, seed):
    """Every named kind and matrices of 1..6 targets, 0..n - k controls, on random qubits."""
    rng = np.random.default_rng(seed)
    names = [g for g in W.GATE_NAMES if g != "matrix"]
    gates = []
    for i in range(count):
        if i % 3 == 2:
            k = int(rng.integers(1, min(6, n) + 1))
            c = int(rng.integers(0, min(n - k, 8) + 1)) if rng.random() < 0.4 else 0
            qs = [int(q) for q in rng.choice(n, size=k + c, replace=False)]
            gates.append(W.Gate("matrix", tuple(qs[:k]), tuple(qs[k:]), (), W.haar_unitary(rng, 1 << k)))
        else:
            name = names[int(rng.integers(0, len(names)))]
            c = int(rng.integers(0, min(n - 1, 2) + 1))
            qs = [int(q) for q in rng.choice(n, size=1 + c, replace=False)]
            gates.append(W.Gate(name, (qs[0],), tuple(qs[1:]),
                                tuple(float(x) for x in rng.uniform(0, 6.28, W.N_PARAMS[name]))))
    return gates


def run(h, n, dtype, gates, opts, timed=False):
    B.sv_reset(h)
    B.sv_profile_enable(h, timed)
    st = B.sv_apply_circuit(h, gates, opts)
    B.sv_profile_enable(h, False)
    recs = B.sv_profile_read(h)
    assert len(recs) == (st["sweeps"] if timed else 0)
    return st, B.sv_copy_to_host(h, n, dtype).astype(np.complex128)


# 13 / 12 (complex64 / complex128): the largest states; 14 / 13: launches per sweep
@pytest.mark.parametrize("dtype", DTYPES, ids=IDS)
@pytest.mark.parametrize("n", [1, 2, 3, 7, 8, 9, 10, 11, 12, 13, 14])
def test_steps_match_oracle_and_launches(dtype, n):
    gates = mixed_gates(n, 60, 100 + n)
    want = oracle.run(gates, n)
    h = B.sv_create(n, dtype)
    try:
        for mode, k in [(B.SV_PLAN_PLAIN, 5), (B.SV_PLAN_PASSES, 4)] + [(B.SV_PLAN_GREEDY, k) for k in range(1, 7)]:
            opts = B.make_opts(mode, k)
            st, got = run(h, n, dtype, gates, opts)
            st2, ref = run(h, n, dtype, gates, opts, timed=True)
            assert st == st2
            assert float(np.max(np.abs(got - want))) <= TOL[dtype]
            assert float(np.max(np.abs(got - ref))) <= TOL[dtype]
    finally:
        B.sv_destroy(h)


@pytest.mark.parametrize("dtype", DTYPES, ids=IDS)
def test_calls_in_a_row_and_long_programs(dtype):
    """More calls than program slots without a wait between them, a circuit of
    more steps than the table holds at a time, one too long for a slot, and a
    relaid-out state."""
    n = 11
    h = B.sv_create(n, dtype)
    try:
        B.sv_swap_bits(h, 1, 6, 4)
        gates = []
        for i in range(9):
            part = mixed_gates(n, 5 + i, i)
            gates += part
            B.sv_apply_circuit(h, part, B.make_opts(B.SV_PLAN_PLAIN))
        for seed in (1, 2):
            part = W.layered_u3_pairing(n, 13, seed, "cx_or_cz")  # 208 one-target steps
            gates += part
            B.sv_apply_circuit(h, part, B.make_opts(B.SV_PLAN_PLAIN))
        got = B.sv_copy_to_host(h, n, dtype).astype(np.complex128)
        assert float(np.max(np.abs(got - oracle.run(gates, n)))) <= 4 * TOL[dtype]
        part = W.layered_u3_pairing(n, 60, 3, "cx_or_cz")  # 960 steps: beyond a slot
        st, got = run(h, n, dtype, part, B.make_opts(B.SV_PLAN_PLAIN))
        assert st["sweeps"] == len(part)
        assert float(np.max(np.abs(got - oracle.run(part, n)))) <= 5 * TOL[dtype]
    finally:
        B.sv_destroy(h)


def test_captured_circuit_replays():
    """A stream being captured records the launches themselves: the replay
    does not depend on later calls of the handle."""
    import torch

    import paper_2511_14664_amd as svm

    n = 9
    first, other = W.layered_u3_pairing(n, 4, 4, "cx_or_cz"), W.layered_u3_pairing(n, 4, 5, "cx")
    want1, want2 = oracle.run(first, n), oracle.run(first + other, n)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        s = svm.StateVector(n, B.SV_C128, stream=stream)
        stream.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            s.reset()
            s.apply_circuit(first)
        for _ in range(3):
            g.replay()
            stream.synchronize()
            assert float(np.max(np.abs(s.to_host() - want1))) <= 1e-12
            s.apply_circuit(other)
            assert float(np.max(np.abs(s.to_host() - want2))) <= 1e-12
        s.close()
