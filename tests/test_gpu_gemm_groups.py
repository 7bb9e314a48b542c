"""Products above 128 slots: no waits up to 224 slots, and two slot groups above
256, whose workgroups share out the row tiles unevenly: a tile that two of them
compute is one chain of sums in order of k, continued from memory, so that

  * a user's logits do not depend on which group, tile or packed remainder its
    slots fall into (two users of the same prefix, keys, values and tokens, the
    first and the last of the batch, get the same bits);
  * computing every shared tile whole, which is what a workgroup does whose
    predecessor is late (forced by the wait limit of zero polls), gives the same
    bits, leaves the counters at zero and is no error;
  * two batches in flight on two streams equal each one alone.

The one-layer Qwen3-32B shape takes the split counts of the full model (QKV 5,
O 8, down 10, gate/up unsplit); 300, 359 and 400 slots are the three group
widths (five, six and eight 32-slot tiles) with a last tile of 12, 7 and 16
slots.  tiny-wide-ffn: 160 gate/up row tiles of four k chunks."""
import dataclasses

import numpy as np
import pytest
import torch

import workload as wl
from gpu_harness import load_synthetic_kv, make_verifier
from workload.device import DeviceWeights, kv_rows

pytestmark = pytest.mark.gpu

ONE = dataclasses.replace(wl.MODELS["qwen3-32b"], name="qwen3-32b-one-layer", n_layers=1, vocab=4096)


def _pass(v, w, n, b, drafts, stream=None, graph=False):
    v.verify(n, w.assign, w.draft_len, drafts, None, "greedy", stream=stream, graph=graph)


def _result(v, w, n, b, stream=None):
    lg = v.logits(n, b.T, stream=stream)
    n_acc, tok = v.accept(n, w.n_users)
    torch.cuda.synchronize()
    return n_acc[b.users].copy(), tok[b.users].copy(), lg.cpu().numpy()


def _same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("model,T", [("qwen3-32b-one-layer", 300), ("qwen3-32b-one-layer", 359),
                                     ("qwen3-32b-one-layer", 400), ("tiny-wide-ffn", 359)])
def test_logits_do_not_depend_on_the_slot_group(monkeypatch, model, T):
    monkeypatch.setitem(wl.MODELS, ONE.name, ONE)
    twin = 6                      # drafts of the first and the last user
    left = T - 2 * (twin + 1)
    L = [twin] + [12] * (left // 13) + ([left % 13 - 1] if left % 13 > 1 else []) + [twin]
    if left % 13 == 1:
        L[1] += 1
    P = [20 + (31 * i) % 90 for i in range(len(L))]
    P[-1] = P[0]
    w = wl.custom_workload(model, P, L, seed=31)
    dw = DeviceWeights(w.model, w.seed, gamma="uniform")
    v = make_verifier(w, dw)
    load_synthetic_kv(v, w)
    b = w.batch(0)
    assert b.T == T
    root, drafts = b.root.copy(), b.drafts.copy()
    last = len(L) - 1
    root[last] = root[0]
    drafts[-twin:] = drafts[:twin]
    for l in range(w.model.n_layers):
        k, vv = kv_rows(w.model, w.seed, l, 0, P[0])
        v.write_kv(last, l, 0, k, vv)
        torch.cuda.synchronize()
    for u in range(w.n_users):
        v.reset_user(u, P[u], int(root[u]))
    d = torch.from_numpy(np.ascontiguousarray(drafts)).cuda()
    _pass(v, w, 0, b, d)
    ref = _result(v, w, 0, b)
    assert np.array_equal(ref[2][:twin + 1], ref[2][-(twin + 1):])
    for limit in (0, 0, -1):
        v.wait_limit(limit)
        _pass(v, w, 0, b, d)
        assert _same(_result(v, w, 0, b), ref), limit
    v.close()


@pytest.mark.parametrize("T", [144, 176, 208, 224])
def test_no_waits_up_to_224_slots(T):
    """A gate/up product of more than half and fewer than all CUs' row tiles is
    not split there: the pass does not depend on the wait limit."""
    L = [11] * (T // 12) + ([T % 12 - 1] if T % 12 else [])
    w = wl.custom_workload("tiny-wide-ffn", [(29 * i) % 80 for i in range(len(L))], L, seed=37)
    dw = DeviceWeights(w.model, w.seed)
    v = make_verifier(w, dw)
    load_synthetic_kv(v, w)
    b = w.batch(0)
    assert b.T == T
    for i, u in enumerate(b.users):
        v.reset_user(int(u), int(b.prefix_len[i]), int(b.root[i]))
    d = torch.from_numpy(np.ascontiguousarray(b.drafts)).cuda()
    _pass(v, w, 0, b, d)
    ref = _result(v, w, 0, b)
    v.wait_limit(0)
    _pass(v, w, 0, b, d)
    assert _same(_result(v, w, 0, b), ref)
    v.close()


@pytest.mark.parametrize("graph", [False, True])
def test_batches_on_two_streams(graph):
    prefix = [int(x) for x in np.random.default_rng(6).integers(0, 300, 50)]
    w = wl.custom_workload("tiny-wide-ffn", prefix, [11] * 50, seed=29, assign=[i % 2 for i in range(50)])
    dw = DeviceWeights(w.model, w.seed)
    v = make_verifier(w, dw)
    load_synthetic_kv(v, w)
    batches = [w.batch(n) for n in range(2)]
    assert [b.T for b in batches] == [300, 300]
    devs = []
    for b in batches:
        for i, u in enumerate(b.users):
            v.reset_user(int(u), int(b.prefix_len[i]), int(b.root[i]))
        devs.append(torch.from_numpy(np.ascontiguousarray(b.drafts)).cuda())
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    refs = []
    for n, b in enumerate(batches):
        _pass(v, w, n, b, devs[n], streams[0])
        refs.append(_result(v, w, n, b, streams[0]))
    for rep in range(4):
        v.wait_limit(0 if rep == 2 else -1)
        for n, b in enumerate(batches):
            _pass(v, w, n, b, devs[n], streams[n], graph)
        for n, b in enumerate(batches):
            assert _same(_result(v, w, n, b, streams[n]), refs[n]), (rep, n)
    v.close()
