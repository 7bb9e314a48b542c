"""The fp32 configuration on shapes that leave remainders everywhere: widths
off the 16-column tiles and the 4-element loads, heads of 10 to 128 dims (one
and two dims a lane), contexts around the 16-token pages and the 64- and
256-token blocks of the attention, slot counts around the 16-slot tiles; against
the oracle (bound: 1e-4 of the row's largest logit, the fp32 model's)."""
import dataclasses

import numpy as np
import pytest

import oracle
import workload as wl
from gpu_harness import (assert_decisions, compare_decisions, load_synthetic_kv, logit_rel_err, make_verifier,
                         run_gpu, run_oracle)
from workload.device import DeviceWeights

pytestmark = pytest.mark.gpu

BASE = wl.MODELS["tiny-qknorm"]
SHAPES = {  # d, query heads, KV heads, head_dim, ffn, vocab
    "odd": (36, 3, 1, 10, 77, 101),
    "pairs": (64, 4, 2, 30, 66, 258),
    "wide-head": (68, 2, 1, 128, 130, 515),
    "head-72": (132, 6, 3, 72, 260, 1027),
}
CONTEXTS = {
    "short": ([0, 1, 14], [1, 2, 3]),
    "pages": ([15, 16, 17, 47, 48], [1, 1, 4, 1, 5]),
    "blocks": ([60, 61, 62, 63, 64, 250, 253, 255, 256, 319, 320, 600], [1, 2, 3, 1, 1, 5, 2, 1, 1, 1, 3, 4]),
}


@pytest.mark.parametrize("ctx", list(CONTEXTS))
@pytest.mark.parametrize("shape", list(SHAPES))
def test_f32_shapes(monkeypatch, shape, ctx):
    d, hq, hkv, hd, F, V = SHAPES[shape]
    m = dataclasses.replace(BASE, name="f32-" + shape, d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd,
                            d_ffn=F, vocab=V)
    monkeypatch.setitem(wl.MODELS, m.name, m)
    prefix, L = CONTEXTS[ctx]
    w = wl.custom_workload(m.name, prefix, L, seed=61, q_sigma=1.0)
    dw = DeviceWeights(m, w.seed, gamma="uniform")
    v = make_verifier(w, dw)
    load_synthetic_kv(v, w)
    b = w.batch(0)
    gpu = run_gpu(v, w, 0, b, "stochastic", seed=5, round_=2)
    rl, ref = run_oracle(w, b, "stochastic", seed=5, round_=2, weights=oracle.WeightSource(m, w.seed, "uniform"))
    err = float(logit_rel_err(gpu.logits, rl).max())
    assert err < 1e-4, err
    chk = compare_decisions(gpu.n_acc, gpu.token, ref, b.draft_len, "stochastic", b.drafts, gpu.logits, rl)
    assert_decisions(chk, f"{shape}/{ctx} (err {err:.1e})", end_to_end=True)
    v.close()
