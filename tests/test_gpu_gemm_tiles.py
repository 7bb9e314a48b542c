"""Every tile shape of the 32x32 GEMM form on toy bf16 models, against the
oracle: one to five 32-slot tiles on four waves, six and eight on eight, two
slot groups above 256 slots; both sides of every boundary, and last tiles that
hold at most 16 slots (both planes in one tile) next to ones that hold more.

tiny-wide-ffn: 160 gate/up row tiles, unsplit up to 224 slots, split over every
CU at 225-256 and, at two slot groups, shared out over every CU.
tiny-deep-ffn: a down projection of four row tiles over a k of 16384, split
64 ways (the split-K form at small slot counts), and 128 gate/up row tiles
split in two with a reduction kernel.

Bound: the bf16 model's logits within 1e-3 of the row's largest (activations
carry about 16 bits, new keys and values 8; ten times what these models show).
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

DEEP = dataclasses.replace(wl.MODELS["tiny-bf16"], name="tiny-deep-ffn", n_layers=1, d_model=1024, d_ffn=16384)
SMALL = [2, 16, 17, 32, 33, 48, 49, 64, 65, 80, 96]
LARGE = [129, 144, 160, 161, 176, 192, 193, 208, 288, 304, 320, 321, 336, 384, 385, 400, 416]


def _draft_lengths(T):
    """Draft lengths of users whose slots add up to T (l + 1 slots each)."""
    out = []
    while T > 0:
        n = T if T <= 13 else (7 if T - 7 >= 2 else 5)
        out.append(n - 1)
        T -= n
    return out


@pytest.mark.parametrize("model,T", [("tiny-wide-ffn", T) for T in SMALL + LARGE] +
                                    [("tiny-deep-ffn", T) for T in SMALL + [100, 128, 150]])
def test_tiles_against_oracle(monkeypatch, model, T):
    monkeypatch.setitem(wl.MODELS, "tiny-deep-ffn", DEEP)
    L = _draft_lengths(T)
    prefix = [(37 * i) % 70 for i in range(len(L))]
    w = wl.custom_workload(model, prefix, L, seed=900, q_sigma=1.0)
    dw = DeviceWeights(w.model, w.seed, gamma="uniform")
    v = make_verifier(w, dw)
    load_synthetic_kv(v, w)
    b = w.batch(0)
    assert b.T == T
    gpu = run_gpu(v, w, 0, b, "stochastic", seed=4, round_=1)
    again = run_gpu(v, w, 0, b, "stochastic", seed=4, round_=1)
    rl, ref = run_oracle(w, b, "stochastic", seed=4, round_=1, weights=oracle.WeightSource(w.model, w.seed, "uniform"))
    err = float(logit_rel_err(gpu.logits, rl).max())
    assert err < 1e-3, err
    assert np.array_equal(gpu.logits, again.logits)  # sums are taken in a fixed order
    chk = compare_decisions(gpu.n_acc, gpu.token, ref, b.draft_len, "stochastic", b.drafts, gpu.logits, rl)
    assert_decisions(chk, f"{model}/T={T} (err {err:.1e})", end_to_end=True)
    v.close()
