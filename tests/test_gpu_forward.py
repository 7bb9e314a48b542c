"""End-to-end parity of the GPU verify pass with the oracle on small models:
logits within tolerance, decisions bit-exact outside the window that the
logit tolerance admits, KV append and commit semantics."""
import numpy as np
import pytest
import torch

import oracle
import workload as wl
from paper_2604_20919_amd import sdverify as sdv
from gpu_harness import (assert_decisions, compare_decisions, gpu_prefill, load_synthetic_kv,
                         logit_rel_err, make_verifier, run_gpu, run_oracle)
from workload.device import DeviceWeights, batch_to_device

pytestmark = pytest.mark.gpu


def _check(w, b, gpu, ref_logits, ref, tol, label, mode):
    err = logit_rel_err(gpu.logits, ref_logits)
    print(f"{label}: logit rel err max {err.max():.3e} mean {err.mean():.3e}")
    assert err.max() < tol, f"{label}: logit error {err.max()}"
    chk = compare_decisions(gpu.n_acc, gpu.token, ref, b.draft_len, mode, b.drafts, gpu.logits, ref_logits)
    assert_decisions(chk, label, end_to_end=True)


@pytest.mark.parametrize("model", ["tiny", "tiny-qknorm"])
def test_fp32_model_synthetic_kv(model):
    w = wl.custom_workload(model, [64, 96, 112, 128, 0, 300], [1, 2, 3, 4, 2, 6], seed=31,
                           accept_u_input=True)
    dw = DeviceWeights(w.model, w.seed, gamma="uniform")
    v = make_verifier(w, dw)
    load_synthetic_kv(v, w)
    b = w.batch(0)
    ws = oracle.WeightSource(w.model, w.seed, "uniform")
    for mode in ("stochastic", "greedy"):
        gpu = run_gpu(v, w, 0, b, mode, seed=3, round_=1)
        rl, ref = run_oracle(w, b, mode, seed=3, round_=1, weights=ws)
        _check(w, b, gpu, rl, ref, 1e-4, f"{model}/{mode}", mode)
    v.close()


@pytest.mark.parametrize("gamma", ["ones", "uniform"])
def test_bf16_model_synthetic_kv(gamma):
    # 8 query heads per KV head and 128-wide heads (the 32B head layout);
    # prefixes span several attention chunks, include an empty prefix, and
    # draft lengths give up to 104 query rows per KV head (two row passes)
    w = wl.custom_workload("tiny-bf16", [40, 700, 0, 17, 1030, 255], [1, 7, 3, 12, 4, 2], seed=32,
                           q_sigma=1.0)
    dw = DeviceWeights(w.model, w.seed, gamma=gamma)
    v = make_verifier(w, dw)
    load_synthetic_kv(v, w)
    b = w.batch(0)
    ws = oracle.WeightSource(w.model, w.seed, gamma)
    for mode in ("stochastic", "greedy", "force"):
        gpu = run_gpu(v, w, 0, b, mode, seed=9, round_=2)
        rl, ref = run_oracle(w, b, mode, seed=9, round_=2, weights=ws)
        _check(w, b, gpu, rl, ref, 2e-2, f"tiny-bf16/{gamma}/{mode}", mode)
    v.close()


def _compare_kv(v, m, users, explicit, tol=1e-4):
    for u in users:
        K, V = explicit[u]
        P = K.shape[1]
        for l in range(m.n_layers):
            kd = torch.empty((P, m.n_kv_heads, m.head_dim), dtype=torch.float32, device="cuda")
            vd = torch.empty_like(kd)
            v.read_kv(u, l, 0, kd, vd)
            ek = np.abs(kd.cpu().numpy().reshape(P, -1) - K[l]).max() / np.abs(K[l]).max()
            ev = np.abs(vd.cpu().numpy().reshape(P, -1) - V[l]).max() / np.abs(V[l]).max()
            assert ek < tol and ev < tol, (u, l, ek, ev)


def test_fp32_prefill_via_force_mode_matches_oracle_prefill():
    """Build the cache on the GPU by teacher-forced verify calls with commit
    (chunks of up to 17 tokens), then verify drafts on top; the oracle builds
    its cache with one causal forward.  Logits and KV must agree."""
    m = wl.MODELS["tiny-qknorm"]
    w = wl.custom_workload("tiny-qknorm", [0, 0], [16, 16], seed=33)
    dw = DeviceWeights(m, w.seed, gamma="uniform")
    v = make_verifier(w, dw, extra_ctx=80)
    rng = np.random.default_rng(7)
    P = [45, 70]
    toks = [rng.integers(0, m.vocab, size=P[u] + 1).astype(np.int32) for u in range(2)]
    for u in range(2):
        gpu_prefill(v, u, toks[u], 2, chunk=17)
    ws = oracle.WeightSource(m, w.seed, "uniform")
    explicit = {u: oracle.prefill(m, ws, toks[u][:P[u]]) for u in range(2)}
    _compare_kv(v, m, range(2), explicit)
    # verify drafts on top of the prefilled caches
    w2 = wl.custom_workload("tiny-qknorm", P, [3, 5], seed=34)
    b = w2.batch(0)
    b.root[:] = [toks[0][P[0]], toks[1][P[1]]]
    drafts, q, _ = batch_to_device(b)
    v.verify(0, w2.assign, w2.draft_len, drafts, q, "stochastic", 5, 0)
    gl = v.logits(0, b.T).cpu().numpy()
    n_acc, tok = v.accept(0, 2)
    kvs = oracle.KVSource(m, 0, [0, 1], P, explicit=explicit)
    rl, ref = run_oracle(w2, b, "stochastic", 5, 0, kv=kvs, weights=ws)
    err = logit_rel_err(gl, rl)
    assert err.max() < 1e-4, err.max()
    assert_decisions(compare_decisions(n_acc, tok, ref, b.draft_len, "stochastic", b.drafts, gl, rl),
                     "prefilled fp32 caches", end_to_end=True)
    v.close()


def test_tiny_workload_as_defined():
    """The tiny verify workload exactly as defined: the 2-layer fp32 model
    (d 256, 4/2 heads, hd 64, FFN 512, RoPE base 1e4, V 1024, no QK-norm,
    weights N(0, 0.02), gains 1), 4 users whose caches hold real prefixes of
    {64, 96, 112, 128} uniform token ids, draft lengths {1, 2, 3, 4}, drafts
    drawn from q = softmax(N(0, 1) logits), accept uniforms from the seed.
    The GPU builds the caches by teacher-forced verify calls, the oracle by
    one causal forward per user; the caches agree, and the verify pass
    agrees in all three modes (logits to 1e-4 relative, decisions exact
    outside the counted window)."""
    w = wl.workload("tiny")
    m = w.model
    assert list(w.prefix_len) == [64, 96, 112, 128] and list(w.draft_len) == [1, 2, 3, 4]
    dw = DeviceWeights(m, w.seed)
    v = make_verifier(w, dw, max_draft=15, max_batch_tokens=16)
    b = w.batch(0)
    assert b.accept_u is not None
    ws = oracle.WeightSource(m, w.seed)
    explicit = {}
    for i, u in enumerate(b.users):
        toks = np.concatenate([wl.prefix_tokens(w, int(u)), [b.root[i]]]).astype(np.int32)
        gpu_prefill(v, int(u), toks, w.n_users)
        assert v.user_state(int(u)) == (int(b.prefix_len[i]), int(b.root[i]))
        explicit[int(u)] = oracle.prefill(m, ws, toks[:-1])
    _compare_kv(v, m, [int(u) for u in b.users], explicit)
    kvs = oracle.KVSource(m, 0, b.users, b.prefix_len, explicit=explicit)
    for mode in ("stochastic", "greedy", "force"):
        gpu = run_gpu(v, w, 0, b, mode, seed=w.seed, round_=0)
        rl, ref = run_oracle(w, b, mode, seed=w.seed, round_=0, kv=kvs, weights=ws)
        _check(w, b, gpu, rl, ref, 1e-4, f"tiny workload/{mode}", mode)
        if mode == "force":
            assert np.array_equal(gpu.n_acc, b.draft_len)
    v.close()


def test_commit_advances_users_and_rounds_compose():
    """Two rounds with commit: round 2 of the GPU path equals the oracle's
    round 2 computed on the oracle's own round-1 result."""
    m = wl.MODELS["tiny"]
    w = wl.custom_workload("tiny", [20, 33, 5], [3, 2, 4], seed=35)
    dw = DeviceWeights(m, w.seed, gamma="uniform")
    v = make_verifier(w, dw, extra_ctx=16)
    load_synthetic_kv(v, w)
    b = w.batch(0)
    ws = oracle.WeightSource(m, w.seed, "uniform")
    gpu = run_gpu(v, w, 0, b, "greedy", commit=True)
    rl, ref = run_oracle(w, b, "greedy", weights=ws)
    assert np.array_equal(gpu.n_acc, ref["n_acc"]) and np.array_equal(gpu.token, ref["token"])
    for i, u in enumerate(b.users):
        P, root = v.user_state(int(u))
        assert P == b.prefix_len[i] + 1 + ref["n_acc"][i] and root == ref["token"][i]
    # the oracle's cache after round 1: synthetic prefix + the committed slots
    _, K1, V1 = oracle.forward(m, ws, oracle.KVSource(m, w.seed, b.users, b.prefix_len),
                               b.prefix_len, b.n_slots, b.slot_tokens(), want_kv=True)
    explicit = {}
    off = 0
    for i, u in enumerate(b.users):
        P0 = int(b.prefix_len[i])
        keep = 1 + int(ref["n_acc"][i])
        Kp = np.zeros((m.n_layers, P0 + keep, m.n_kv_heads * m.head_dim), np.float32)
        Vp = np.zeros_like(Kp)
        for l in range(m.n_layers):
            kk = np.empty((P0, m.n_kv_heads, m.head_dim), np.float32)
            vv = np.empty_like(kk)
            wl.fill_kv(m, w.seed, l, int(u), 0, kk)
            wl.fill_kv(m, w.seed, l, int(u), 1, vv)
            Kp[l, :P0] = kk.reshape(P0, -1)
            Vp[l, :P0] = vv.reshape(P0, -1)
            Kp[l, P0:] = K1[l, off:off + keep]
            Vp[l, P0:] = V1[l, off:off + keep]
        explicit[int(u)] = (Kp, Vp)
        off += int(b.n_slots[i])
    P2 = [int(b.prefix_len[i]) + 1 + int(ref["n_acc"][i]) for i in range(len(b.users))]
    w2 = wl.custom_workload("tiny", P2, [2, 4, 1], seed=36)
    b2 = w2.batch(0)
    b2.root[:] = ref["token"]
    drafts, q, _ = batch_to_device(b2)
    v.verify(0, w2.assign, w2.draft_len, drafts, q, "greedy")
    gl = v.logits(0, b2.T).cpu().numpy()
    n2, t2 = v.accept(0, 3)
    rl2, ref2 = run_oracle(w2, b2, "greedy", kv=oracle.KVSource(m, 0, b2.users, P2, explicit=explicit),
                           weights=ws)
    assert logit_rel_err(gl, rl2).max() < 1e-4
    assert np.array_equal(n2, ref2["n_acc"]) and np.array_equal(t2, ref2["token"])
    v.close()


def test_determinism_two_runs_bit_identical():
    w = wl.custom_workload("tiny-bf16", [300, 12, 77], [4, 9, 2], seed=37)
    dw = DeviceWeights(w.model, w.seed)
    v = make_verifier(w, dw)
    load_synthetic_kv(v, w)
    b = w.batch(0)
    a = run_gpu(v, w, 0, b, "stochastic", seed=1)
    c = run_gpu(v, w, 0, b, "stochastic", seed=1)
    assert np.array_equal(a.logits, c.logits)
    assert np.array_equal(a.n_acc, c.n_acc) and np.array_equal(a.token, c.token)
    v.close()


def _ragged_draft_lengths(T_target, rng):
    """Draft lengths 1..12 whose slot total (l + 1 per user) is T_target."""
    L, T = [], 0
    while T < T_target:
        rem = T_target - T
        if rem == 1:
            # one slot left: an earlier user drafts one more token
            j = next(i for i, x in enumerate(L) if x < 12)
            L[j] += 1
            T += 1
            continue
        l = int(min(rng.integers(1, 13), rem - 1))
        L.append(l)
        T += l + 1
    assert T == T_target
    return L


@pytest.mark.parametrize("T_target", [17, 64, 65, 70, 75, 80, 96, 97, 105, 112, 113, 120, 128, 129, 150, 224, 225,
                                      232, 240, 241, 250, 256, 257, 300, 320, 321, 416])
def test_bf16_every_gemm_tile_class(T_target):
    """Query-slot totals around every boundary between the GEMM tile classes of
    the toy model: the 16x16 form up to 96 slots, the 32x32 form above (four
    and five 32-slot tiles on four waves, six and eight on eight, two slot
    groups above 256 slots; up to 256 a last tile of at most 16 slots holds
    both their planes), split-K and unsplit paths, up to the 416-slot
    maximum."""
    rng = np.random.default_rng(T_target)
    L = _ragged_draft_lengths(T_target, rng)
    prefix = [int(p) for p in rng.integers(0, 200, size=len(L))]
    w = wl.custom_workload("tiny-bf16", prefix, L, seed=40 + T_target, q_sigma=1.0)
    dw = DeviceWeights(w.model, w.seed, gamma="uniform")
    v = make_verifier(w, dw)
    load_synthetic_kv(v, w)
    b = w.batch(0)
    assert b.T == T_target
    ws = oracle.WeightSource(w.model, w.seed, "uniform")
    gpu = run_gpu(v, w, 0, b, "stochastic", seed=2, round_=3)
    rl, ref = run_oracle(w, b, "stochastic", seed=2, round_=3, weights=ws)
    _check(w, b, gpu, rl, ref, 2e-2, f"tiny-bf16/T={b.T}", "stochastic")
    v.close()


@pytest.mark.parametrize("T_target", [17, 40, 96])
def test_last_split_gate_up_repeats_and_never_waits(T_target):
    """Below 97 slots the toy bf16 model's gate/up product (16 row tiles of
    128 rows) is split over k in four, and whichever split of a tile counts
    last adds the others' sums in split order and applies SwiGLU.  Parity
    with the oracle; a second pass bit-identical to the first (the tile
    counters came back to zero, the sum order does not depend on which
    split comes last); and with the stream-K wait bound at zero polls the
    pass still succeeds, since this form never waits."""
    rng = np.random.default_rng(400 + T_target)
    L = _ragged_draft_lengths(T_target, rng)
    prefix = [int(p) for p in rng.integers(0, 300, size=len(L))]
    w = wl.custom_workload("tiny-bf16", prefix, L, seed=130 + T_target, q_sigma=1.0)
    dw = DeviceWeights(w.model, w.seed, gamma="uniform")
    v = make_verifier(w, dw)
    load_synthetic_kv(v, w)
    b = w.batch(0)
    assert b.T == T_target
    gpu = run_gpu(v, w, 0, b, "stochastic", seed=4, round_=1)
    rl, ref = run_oracle(w, b, "stochastic", seed=4, round_=1, weights=oracle.WeightSource(w.model, w.seed, "uniform"))
    _check(w, b, gpu, rl, ref, 2e-2, f"tiny-bf16/T={b.T}", "stochastic")
    again = run_gpu(v, w, 0, b, "stochastic", seed=4, round_=1)
    assert np.array_equal(again.logits, gpu.logits)
    assert np.array_equal(again.n_acc, gpu.n_acc) and np.array_equal(again.token, gpu.token)
    v.wait_limit(0)
    bounded = run_gpu(v, w, 0, b, "stochastic", seed=4, round_=1)
    v.wait_limit(-1)
    assert np.array_equal(bounded.logits, gpu.logits)
    v.close()


@pytest.mark.parametrize("T_target", [40, 120])
def test_split_gate_up_with_reduction_kernel(T_target):
    """A gate/up product of 96 row tiles of 256 rows (a 12288-wide
    feed-forward layer) is split over k in two, and a separate kernel adds
    the halves and applies SwiGLU: the form for products too wide for the
    16x16 tiles and too narrow to fill the CUs unsplit.  Parity with the
    oracle."""
    rng = np.random.default_rng(300 + T_target)
    L = _ragged_draft_lengths(T_target, rng)
    prefix = [int(p) for p in rng.integers(0, 300, size=len(L))]
    w = wl.custom_workload("tiny-mid-ffn", prefix, L, seed=110 + T_target, q_sigma=1.0)
    dw = DeviceWeights(w.model, w.seed, gamma="uniform")
    v = make_verifier(w, dw)
    load_synthetic_kv(v, w)
    b = w.batch(0)
    assert b.T == T_target
    gpu = run_gpu(v, w, 0, b, "stochastic", seed=4, round_=1)
    rl, ref = run_oracle(w, b, "stochastic", seed=4, round_=1, weights=oracle.WeightSource(w.model, w.seed, "uniform"))
    _check(w, b, gpu, rl, ref, 2e-2, f"tiny-mid-ffn/T={b.T}", "stochastic")
    v.close()


@pytest.mark.parametrize("T_target", [225, 240, 256])
def test_split_gate_up_over_all_cus(T_target):
    """At 225..256 slots a gate/up product of more than 128 and fewer than
    256 row tiles is split over one workgroup per CU, each taking an equal
    run of (tile, k-chunk) pairs; a tile's last workgroup adds the partial
    sums the earlier ones left and applies SwiGLU.  Parity with the oracle
    on a model whose 20480-wide feed-forward layer takes that form, then the
    error path of the bounded wait: a limit of zero polls makes the pass
    report a device error without committing, and the pass after it (limit
    restored) is bit-identical to the first, so the tile counters came back
    to zero."""
    rng = np.random.default_rng(100 + T_target)
    L = _ragged_draft_lengths(T_target, rng)
    prefix = [int(p) for p in rng.integers(0, 300, size=len(L))]
    w = wl.custom_workload("tiny-wide-ffn", prefix, L, seed=70 + T_target, q_sigma=1.0)
    dw = DeviceWeights(w.model, w.seed, gamma="uniform")
    v = make_verifier(w, dw)
    load_synthetic_kv(v, w)
    b = w.batch(0)
    assert b.T == T_target
    ws = oracle.WeightSource(w.model, w.seed, "uniform")
    gpu = run_gpu(v, w, 0, b, "stochastic", seed=4, round_=1)
    rl, ref = run_oracle(w, b, "stochastic", seed=4, round_=1, weights=ws)
    _check(w, b, gpu, rl, ref, 2e-2, f"tiny-wide-ffn/T={b.T}", "stochastic")

    state = [v.user_state(int(u)) for u in b.users]
    v.wait_limit(0)
    drafts, q, au = batch_to_device(b)
    v.verify(0, w.assign, w.draft_len, drafts, q, "stochastic", 4, 1, au)
    with pytest.raises(sdv.SdError) as e:
        v.accept(0, w.n_users, True)
    assert e.value.status == sdv.SD_EDEVICE
    assert [v.user_state(int(u)) for u in b.users] == state
    v.wait_limit(-1)
    again = run_gpu(v, w, 0, b, "stochastic", seed=4, round_=1)
    assert np.array_equal(again.logits, gpu.logits)
    assert np.array_equal(again.n_acc, gpu.n_acc) and np.array_equal(again.token, gpu.token)
    v.close()
