"""Attention items of at most two 16-row query tiles, whose four waves share out
the tokens: one tile (four stripes) and two (two stripes), contexts around the
32-token block, the stripes and the length up to which an item is a whole
context, alone and in a batch with users of more rows, against the oracle.

Bound: logits within 1e-3 of the row's largest (activations and probabilities
carry about 16 bits, cached keys and values 8; ten times what this model shows).
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

# two query heads a KV head: one tile up to eight slots
G2 = dataclasses.replace(wl.MODELS["tiny-bf16"], name="tiny-g2", n_q_heads=4, n_kv_heads=2)
CASES = {
    "one-tile": ("tiny-bf16", [0, 1, 30, 31, 61, 62, 126, 127, 200, 511], [1] * 10),
    "two-tiles": ("tiny-bf16", [0, 13, 28, 29, 60, 92, 255, 600], [2, 3, 3, 2, 3, 3, 2, 3]),
    "solo-last": ("tiny-bf16", [158, 124, 5], [1, 3, 2]),          # 160 and 128 tokens
    "split-first": ("tiny-bf16", [159, 125, 5, 128], [1, 3, 2, 1]),  # one token more
    "short": ("tiny-bf16", [3, 29, 100], [1, 1, 2]),
    "longer-first": ("tiny-bf16", [511, 509], [1, 3]),
    "long": ("tiny-bf16", [2300, 1500, 40, 4000], [1, 2, 3, 1]),
    "mixed": ("tiny-bf16", [300, 3, 700, 1400, 129], [1, 12, 3, 4, 2]),
    "g2": ("tiny-g2", [0, 100, 400, 33], [1, 7, 8, 12]),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_few_rows_against_oracle(monkeypatch, case):
    monkeypatch.setitem(wl.MODELS, "tiny-g2", G2)
    model, prefix, L = CASES[case]
    w = wl.custom_workload(model, prefix, L, seed=902, q_sigma=1.0)
    dw = DeviceWeights(w.model, w.seed, gamma="uniform")
    v = make_verifier(w, dw)
    load_synthetic_kv(v, w)
    b = w.batch(0)
    gpu = run_gpu(v, w, 0, b, "stochastic", seed=4, round_=1)
    again = run_gpu(v, w, 0, b, "stochastic", seed=4, round_=1)
    rl, ref = run_oracle(w, b, "stochastic", seed=4, round_=1, weights=oracle.WeightSource(w.model, w.seed, "uniform"))
    err = float(logit_rel_err(gpu.logits, rl).max())
    assert err < 1e-3, err
    assert np.array_equal(gpu.logits, again.logits)  # partials are merged in a fixed order
    chk = compare_decisions(gpu.n_acc, gpu.token, ref, b.draft_len, "stochastic", b.drafts, gpu.logits, rl)
    assert_decisions(chk, f"{case} (err {err:.1e})", end_to_end=True)
    v.close()
