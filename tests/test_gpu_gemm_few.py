"""Few-slot products (at most 16 slots; whole sums in one workgroup, epilogues
in the same launch) on toy bf16 models, against the oracle: both planes in one
operand up to 8 slots and one each above, both sides of the hand-over to the
tiled forms.

few-half: 8-row workgroups (the residual products leave half the CUs idle),
k ranges of 24 and 40 fragments (waves without a share, uneven last steps).
few-whole: 16-row workgroups of the residual products, 512 gate/up workgroups
(two a CU).  few-over: more gate/up workgroups than that, which the tiled
form takes, between products that stay.

Bound: logits within 1e-3 of the row's largest, as for the tiled forms.
"""
import dataclasses

import numpy as np
import pytest

import oracle
import workload as wl
from gpu_harness import (assert_decisions, compare_decisions, load_synthetic_kv, logit_rel_err, make_verifier,
                         run_gpu, run_oracle)
from workload.device import DeviceWeights

pytestmark = pytest.mark.gpu

BASE = wl.MODELS["tiny-bf16"]
MODELS = {
    "few-half": dataclasses.replace(BASE, name="few-half", n_q_heads=6, n_kv_heads=1, d_model=768, d_ffn=1280),
    "few-whole": dataclasses.replace(BASE, name="few-whole", d_model=2560, d_ffn=8192),
    "few-over": dataclasses.replace(BASE, name="few-over", d_model=2304, d_ffn=8448),
}


@pytest.mark.parametrize("lens", [[1], [1, 2], [6], [7], [3, 3], [8], [2, 4, 6], [7, 7], [8, 7]])
@pytest.mark.parametrize("model", sorted(MODELS))
def test_few_slots_against_oracle(monkeypatch, model, lens):
    monkeypatch.setitem(wl.MODELS, model, MODELS[model])
    w = wl.custom_workload(model, [(37 * i) % 70 for i in range(len(lens))], lens, seed=901, q_sigma=1.0)
    dw = DeviceWeights(w.model, w.seed, gamma="uniform")
    v = make_verifier(w, dw)
    load_synthetic_kv(v, w)
    b = w.batch(0)
    gpu = run_gpu(v, w, 0, b, "stochastic", seed=4, round_=1)
    again = run_gpu(v, w, 0, b, "stochastic", seed=4, round_=1)
    rl, ref = run_oracle(w, b, "stochastic", seed=4, round_=1, weights=oracle.WeightSource(w.model, w.seed, "uniform"))
    err = float(logit_rel_err(gpu.logits, rl).max())
    assert err < 1e-3, err
    assert np.array_equal(gpu.logits, again.logits)  # sums are taken in a fixed order
    chk = compare_decisions(gpu.n_acc, gpu.token, ref, b.draft_len, "stochastic", b.drafts, gpu.logits, rl)
    assert_decisions(chk, f"{model}/T={b.T} (err {err:.1e})", end_to_end=True)
    v.close()
