"""The context-free sampler against the oracle on vocabularies and rows where
its chunks and tiles end: odd vocabularies (element loads), one tile, one more
than a tile, many chunks; runs of more than 64 drafts; logits masked to -inf
and to the lowest fp32; rows whose first tiles hold nothing else; ties of the
maximum (the lowest index wins).  Decisions and tokens agree except within the
window of two fp32 evaluations (1e-3 on ratios and race keys)."""
import numpy as np
import pytest
import torch

import oracle
from gpu_harness import assert_decisions, compare_decisions
from paper_2604_20919_amd import sdverify as sv

pytestmark = pytest.mark.gpu

LENS = {"few": [1, 3, 2], "long": [70, 64, 1, 63, 130], "many": [2, 5, 1, 7, 3, 4, 6, 1] * 6}


def _rows(rng, T, V, kind):
    z = (rng.standard_normal((T, V)) * 1.4).astype(np.float32)
    if kind == "masked":
        z[:, rng.random(V) < 0.7] = -np.inf
        z[::2, : V // 2] = np.finfo(np.float32).min
        z[1::2, : V // 2] = -np.inf
        z[:, V - 1] = 3.0  # something stays visible
    elif kind == "ties":
        z = np.round(z * 2) / 2
    return z


@pytest.mark.parametrize("mode", ["stochastic", "greedy"])
@pytest.mark.parametrize("kind", ["plain", "masked", "ties"])
@pytest.mark.parametrize("V,lens", [(3, "long"), (1021, "long"), (4096, "few"), (4097, "many"), (8196, "long"),
                                    (12290, "many"), (50257, "few"), (151936, "few")])
def test_edges(V, lens, kind, mode):
    rng = np.random.default_rng(V * 7 + len(kind))
    L = LENS[lens]
    nd, T = sum(L), sum(L) + len(L)
    z = _rows(rng, T, V, kind)
    # q close to p at most drafts, so that long runs are accepted
    slot = np.concatenate([np.arange(l) + o for l, o in zip(L, np.cumsum([0] + [l + 1 for l in L])[:-1])])
    zq = z[slot].astype(np.float64)
    zq += 0.05 * rng.standard_normal(zq.shape)
    q = np.exp(zq - zq.max(axis=1, keepdims=True))
    q = (q / q.sum(axis=1, keepdims=True)).astype(np.float32)
    drafts = np.array([rng.choice(V, p=r.astype(np.float64) / r.astype(np.float64).sum()) for r in q], np.int32)
    if mode == "greedy":
        drafts = np.where(rng.random(nd) < 0.97, z[slot].argmax(axis=1), drafts).astype(np.int32)
    users = np.sort(rng.choice(1000, len(L), replace=False)).astype(np.int32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    dz, dq, dd = dev(z), dev(q), dev(drafts)
    out = torch.full((2 * len(L) + 1,), -7, dtype=torch.int32, device="cuda")
    sv.sd_sample_logits_noalloc(users, L, V, dd, dq, dz, mode, out, seed=9, round_=4)
    r = out.cpu().numpy()
    assert r[-1] == 0
    ref = oracle.sample(mode, users, L, z, drafts, q, None, 9, 4)
    chk = compare_decisions(r[:len(L)], r[len(L):-1], ref, L, mode)
    assert_decisions(chk, f"V={V} {lens} {kind} {mode}: accepted {int(ref['n_acc'].sum())} of {nd}", end_to_end=False)
