"""The learned planner predicts a pass from the features that the pass is recorded
with when it runs, diagonal steps included: the predicted time of the plan that
runs is that of its records."""
import numpy as np
import pytest

from workloads import Gate

from paper_2511_14664_amd import _binding as B

pytestmark = pytest.mark.gpu


def phase_layers(n, layers):
    """H, then layers of every controlled phase and RX on every qubit."""
    g = [Gate("h", (q,)) for q in range(n)]
    for k in range(layers):
        g += [Gate("p", (b,), (a,), (0.1 + 0.01 * (a + b + k),)) for a in range(n) for b in range(a)]
        g += [Gate("rx", (q,), (), (0.3,)) for q in range(n)]
    return g


@pytest.mark.parametrize("n", [16, 20])
def test_predicted_and_recorded_features_agree(n):
    gates = phase_layers(n, 2)
    # (ranking takes the split products for complex64)
    opts = B.make_opts(B.SV_PLAN_LEARNED, 5, B.SV_PREC_BF16X6)
    info = B.sv_pass_plan_info(n, B.SV_C64, gates, B.make_opts(B.SV_PLAN_PASSES, 5, B.SV_PREC_BF16X6))
    h = B.sv_create(n, B.SV_C64)
    compared = 0
    try:
        for seed in range(12):
            m = B.sv_costmodel_create(seed)
            try:
                chosen, pred = B.sv_costmodel_rank(m, n, B.SV_C64, gates, 5)
                if chosen != 0 or not np.all(np.isfinite(pred)):
                    continue  # this untrained model prefers a greedy plan
                B.sv_set_costmodel(h, m)
                B.sv_reset(h)
                B.sv_profile_enable(h, True)
                B.sv_apply_circuit(h, gates, opts)
                B.sv_profile_enable(h, False)
                raw, count = B.sv_profile_read_raw(h)
                recs = [raw[i] for i in range(count)]
                assert any(r.kind == 7 for r in recs)
                ms = np.exp(B.sv_costmodel_predict(m, B.sv_sweep_features(n, B.SV_C64, raw, count)).astype(np.float64))
                total = float(np.sum(ms * np.array([r.bytes * 1e-9 for r in recs])))
                print(f"n={n} seed {seed}: predicted {pred[5]:.6g}, of the records {total:.6g}, "
                      f"{sum(r.blocks for r in recs)} steps, {info['blocks']} blocks in the default plan", flush=True)
                # both are sums of the same FP32 predictions
                assert abs(total - float(pred[5])) <= 1e-4 * total
                # diagonal steps did run: some pass does fewer operations than its steps as blocks would take
                assert any(r.kind == 7 and r.flops < 0.99 * r.blocks * 126.0 * 2.0 ** n for r in recs)
                compared += 1
            finally:
                B.sv_set_costmodel(h, None)
                B.sv_costmodel_destroy(m)
    finally:
        B.sv_destroy(h)
    assert compared > 0
