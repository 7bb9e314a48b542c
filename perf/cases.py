"""Timed cases of the library: the calls that an edge server and a drafting
device make, each through the public entry points (Verifier and the sd_*
wrappers), over the sizes that those calls are used at.

A case is a dict of plain values:
  call    "verify"  one verification batch: sd_verify_batch[_graph|_sparse] + sd_accept, logits read back
          "draft"   one decode step of a drafting model: sd_draft_batch with its distributions + sd_accept
          "score"   teacher forcing (prompt prefill / scoring): force mode, committed, logits read back
          "sample"  the context-free accept/resample step on given logits: sd_sample_logits_noalloc
          "load"    a prefix entering the paged cache: sd_kv_write of every layer
  model   one of MODELS; layers: decoder layers of the context (the 32B shape runs a quarter of its
          depth so that several contexts fit one card; the 1.7B shape runs whole)
  users, l_lo..l_hi (draft lengths), p_lo..p_hi (cached prefixes); lens: seed of the ragged lengths
Weights are N(0, 0.02), cached keys and values N(0, 1), draft distributions softmax of Gaussian
logits as wide as a random-init target's: the distributions of the repository's own workloads.
"""
from __future__ import annotations

import math
import random
from types import SimpleNamespace

import numpy as np
import torch

from paper_2604_20919_amd import sdverify as sv
from paper_2604_20919_amd.verifier import Verifier

MAX_SLOTS = 416          # most query slots of one bf16 batch
MAX_PREFIX_SUM = 90000   # cached tokens of one batch (bounds a state's memory)
WEIGHT_STD = 0.02


def _shape(n_layers, d_model, n_q_heads, n_kv_heads, head_dim, d_ffn, vocab, rope_base, qk_norm, dtype):
    return SimpleNamespace(n_layers=n_layers, d_model=d_model, n_q_heads=n_q_heads, n_kv_heads=n_kv_heads,
                           head_dim=head_dim, d_ffn=d_ffn, vocab=vocab, rope_base=rope_base, rms_eps=1e-6,
                           qk_norm=qk_norm, dtype=dtype)


MODELS = {
    "qwen3-1.7b": (28, 2048, 16, 8, 128, 6144, 151936, 1e6, True, "bf16"),
    "qwen3-32b": (16, 5120, 64, 8, 128, 25600, 151936, 1e6, True, "bf16"),
    "tiny": (2, 256, 4, 2, 64, 512, 1024, 1e4, False, "f32"),
}


def _case(name, call, model, users, l, p, lens, mode="stochastic", graph=False, sparse=0):
    return {"name": name, "call": call, "model": model, "users": users, "l_lo": l[0], "l_hi": l[1],
            "p_lo": p[0], "p_hi": p[1], "lens": lens, "mode": mode, "graph": graph, "sparse": sparse}


def listed():
    return [
        # a device drafting one token for itself: the smallest call, one query slot
        _case("draft-1.7b-1u", "draft", "qwen3-1.7b", 1, (0, 0), (512, 512), 1),
        # the drafting model serving the paper's largest user count at once
        _case("draft-1.7b-14u", "draft", "qwen3-1.7b", 14, (0, 0), (64, 2048), 2),
        # a small target verified from a graph: the repository's 8-user batch
        _case("verify-1.7b-8u", "verify", "qwen3-1.7b", 8, (1, 8), (512, 512), 3, graph=True),
        # the paper's standard setting, six users on the large target
        _case("verify-32b-6u", "verify", "qwen3-32b", 6, (1, 7), (128, 2048), 4),
        # the repository's 16-user batch, greedy
        _case("verify-32b-16u", "verify", "qwen3-32b", 16, (4, 4), (1024, 1024), 5, mode="greedy"),
        # one batch of the pipelined workload: long contexts, sparse draft rows
        _case("verify-32b-16u-long", "verify", "qwen3-32b", 16, (1, 10), (1024, 8192), 6, sparse=64),
        # the repository's headline: 32 ragged users
        _case("verify-32b-32u", "verify", "qwen3-32b", 32, (1, 12), (256, 4096), 7),
        # a busy server past the headline's slot count
        _case("verify-32b-44u", "verify", "qwen3-32b", 44, (1, 12), (256, 2048), 8),
        # prompts entering by teacher forcing, 64 slots a user: the widest batch
        _case("score-32b-6u", "score", "qwen3-32b", 6, (63, 63), (0, 1024), 9, mode="force"),
        # accept/resample alone, for a program with its own forward pass
        _case("sample-16u", "sample", "qwen3-32b", 16, (1, 8), (0, 0), 10),
        # one user's prefix handed over to the paged cache
        _case("load-32b-4096", "load", "qwen3-32b", 1, (1, 1), (4096, 4096), 11),
        # the fp32 configuration: the repository's tiny workload
        _case("verify-tiny-f32", "verify", "tiny", 4, (1, 4), (64, 128), 12),
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def draw(rng):
    while True:
        lens = rng.randrange(1 << 30)
        kind = rng.choice(["draft", "small", "large", "large", "large", "score", "sample", "load", "f32"])
        p = sorted((_log(rng, 16, 8192), _log(rng, 16, 8192)))
        mode = rng.choice(["stochastic", "stochastic", "greedy"])
        if kind == "draft":
            c = _case("", "draft", "qwen3-1.7b", _log(rng, 1, 40), (0, 0), p, lens, mode)
        elif kind == "small":
            c = _case("", "verify", "qwen3-1.7b", _log(rng, 1, 32), (1, rng.randint(1, 12)), p, lens, mode,
                      graph=rng.random() < 0.5)
        elif kind == "large":
            c = _case("", "verify", "qwen3-32b", _log(rng, 1, 60), (1, rng.randint(1, 12)), p, lens, mode,
                      graph=rng.random() < 0.3)
            if mode == "stochastic" and not c["graph"] and rng.random() < 0.3:
                c["sparse"] = _log(rng, 4, 512)
        elif kind == "score":
            n = rng.randint(7, 63)
            c = _case("", "score", rng.choice(["qwen3-1.7b", "qwen3-32b"]), rng.randint(1, 380 // (n + 1)),
                      (n, n), sorted((rng.randint(0, 1024), rng.randint(0, 1024))), lens, "force")
        elif kind == "sample":
            c = _case("", "sample", "qwen3-32b", _log(rng, 1, 48), (1, rng.randint(1, 12)), (0, 0), lens, mode)
            c["vocab"] = rng.randint(8000, 160000)
        elif kind == "load":
            c = _case("", "load", "qwen3-32b", rng.randint(1, 3), (1, 1), p, lens)
        else:
            c = _case("", "verify", "tiny", _log(rng, 1, 24), (1, rng.randint(1, 8)),
                      sorted((rng.randint(1, 512), rng.randint(1, 512))), lens, mode)
        del c["name"]
        P, L = _lengths(c)
        if sum(L) + len(L) <= 380 and sum(P) <= MAX_PREFIX_SUM:
            return c


# ---------------------------------------------------------------------------
# inputs, made on the GPU from (case, seed)
# ---------------------------------------------------------------------------

def _lengths(c):
    """Prefix and draft length of every user (the case's, whatever the seed)."""
    r = random.Random(c["lens"])
    P = [r.randint(c["p_lo"], c["p_hi"]) for _ in range(c["users"])]
    L = [r.randint(c["l_lo"], c["l_hi"]) for _ in range(c["users"])]
    return P, L


def _gen(seed, *what):
    g = torch.Generator(device="cuda")
    g.manual_seed(random.Random(repr((seed,) + what)).getrandbits(62))
    return g


def _dtype(m):
    return torch.bfloat16 if m.dtype == "bf16" else torch.float32


LAYER_SHAPES = (("wq", lambda m: (m.n_q_heads * m.head_dim, m.d_model)),
                ("wk", lambda m: (m.n_kv_heads * m.head_dim, m.d_model)),
                ("wv", lambda m: (m.n_kv_heads * m.head_dim, m.d_model)),
                ("wo", lambda m: (m.d_model, m.n_q_heads * m.head_dim)),
                ("wg", lambda m: (m.d_ffn, m.d_model)), ("wu", lambda m: (m.d_ffn, m.d_model)),
                ("wd", lambda m: (m.d_model, m.d_ffn)))
GAINS = (("norm1", lambda m: m.d_model), ("norm2", lambda m: m.d_model), ("qnorm", lambda m: m.head_dim),
         ("knorm", lambda m: m.head_dim))


def _normal(n, dt, g, std):
    return torch.empty(n, dtype=dt, device="cuda").normal_(0.0, std, generator=g)


def _layer(m, seed, l):
    """Weights of layer l by name, slices of one buffer, and the gains."""
    g = _gen(seed, "layer", l)
    shapes = [(n, f(m)) for n, f in LAYER_SHAPES]
    flat = _normal(sum(a * b for _, (a, b) in shapes), _dtype(m), g, WEIGHT_STD)
    w, o = {}, 0
    for n, (a, b) in shapes:
        w[n] = flat[o:o + a * b].view(a, b)
        o += a * b
    for n, f in GAINS:
        w[n] = torch.empty(f(m), dtype=torch.float32, device="cuda").uniform_(0.5, 1.5, generator=g).to(_dtype(m))
    return w


def _globals(m, seed):
    g = _gen(seed, "globals")
    w = {n: _normal(m.vocab * m.d_model, _dtype(m), g, WEIGHT_STD).view(m.vocab, m.d_model)
         for n in ("embed", "lm_head")}
    w["norm_f"] = torch.empty(m.d_model, dtype=torch.float32, device="cuda").uniform_(0.5, 1.5, generator=g).to(_dtype(m))
    return w


def _kv(m, seed, l, P):
    """Cached keys and values of layer l, all users' rows one after another."""
    g = _gen(seed, "kv", l)
    kv = _normal(2 * sum(P) * m.n_kv_heads * m.head_dim, _dtype(m), g, 1.0)
    return kv.view(2, sum(P), m.n_kv_heads, m.head_dim)


def _draft_rows(c, V, nd, seed):
    """Draft distributions [nd][V], drafts drawn from them, and the sparse
    rows (listed tokens, probabilities, remainder) when the case has them."""
    g = _gen(seed, "drafts")
    q = torch.empty((nd, V), dtype=torch.float32, device="cuda").normal_(0.0, 1.4, generator=g).softmax(1)
    if c["sparse"]:
        val, idx = q.topk(c["sparse"], dim=1)
        idx, order = idx.sort(dim=1)
        val = val.gather(1, order).contiguous()
        rest = ((1.0 - val.double().sum(1)) / (V - c["sparse"])).float()
        dense = rest[:, None].repeat(1, V).scatter_(1, idx, val)
        drafts = torch.multinomial(dense, 1, generator=g)[:, 0].int()
        return None, drafts, (idx.int().contiguous(), val, rest.contiguous())
    return q, torch.multinomial(q, 1, generator=g)[:, 0].int(), None


def _model(c):
    return _shape(*MODELS[c["model"]])


def _roots(c, m, seed):
    r = random.Random(repr((seed, "roots")))
    return [r.randrange(m.vocab) for _ in range(c["users"])]


def _forced(c, m, seed, nd):
    return torch.randint(0, m.vocab, (nd,), dtype=torch.int32, device="cuda", generator=_gen(seed, "forced"))


def prepare(case, seed):
    c, m = case, _model(case)
    P, L = _lengths(c)
    nd, T, B = sum(L), sum(L) + c["users"], c["users"]
    s = SimpleNamespace(c=c, m=m, P=P, L=L, T=T, B=B, seed=seed & 0xFFFFFFFF)
    if c["call"] == "sample":
        V = c.get("vocab", m.vocab)
        s.V = V
        s.q, s.drafts, _ = _draft_rows(c, V, nd, seed)
        s.logits = torch.empty((T, V), dtype=torch.float32, device="cuda").normal_(0.0, 1.4, generator=_gen(seed, "logits"))
        s.result = torch.empty(2 * B + 1, dtype=torch.int32, device="cuda")
        return s
    glob = _globals(m, seed)
    layers = [_layer(m, seed, l) for l in range(m.n_layers)]
    ptrs = {n: t.data_ptr() for n, t in glob.items()}
    ptrs["layers"] = [{n: t.data_ptr() for n, t in w.items()} for w in layers]
    Lmax = max(1, max(L))
    s.v = Verifier(m, ptrs, n_pages=sum((p + l + 16) // 16 for p, l in zip(P, L)) + 8, max_users=B,
                   max_draft=Lmax, max_batch_users=B, max_batch_tokens=max(2, T),
                   max_ctx=max(p + l for p, l in zip(P, L)) + 2, max_pending=1,
                   logits_out=sv.SD_LOGITS_ALL if c["call"] in ("verify", "score") else sv.SD_LOGITS_AS_NEEDED)
    s.roots = _roots(c, m, seed)
    s.assign, s.L = np.zeros(B, np.int32), np.asarray(L, np.int32)
    if m.dtype == "bf16":  # the packed copies are what the library reads from here on
        glob.pop("lm_head")
        layers = [{n: w[n] for n, _ in GAINS} for w in layers]
    s.keep = (glob, layers)
    off = np.concatenate([[0], np.cumsum(P)])
    if c["call"] == "load":
        s.kv = [_kv(m, seed, l, P) for l in range(m.n_layers)]
        s.off = [int(o) for o in off]
        for u in range(B):
            s.v.reset_user(u, P[u], s.roots[u])
        return s
    for u in range(B):
        s.v.reset_user(u, P[u], s.roots[u])
    for l in range(m.n_layers):
        kv = _kv(m, seed, l, P)
        for u in range(B):
            if P[u]:
                s.v.write_kv(u, l, 0, kv[0, off[u]:off[u + 1]], kv[1, off[u]:off[u + 1]])
    if c["call"] == "draft":
        s.probs = torch.empty((B, m.vocab), dtype=torch.float32, device="cuda")
    elif c["call"] == "score":
        s.drafts = _forced(c, m, seed, nd)
    else:
        s.q, s.drafts, s.sparse = _draft_rows(c, m.vocab, nd, seed)
    s.stream = torch.cuda.Stream() if c["graph"] else None
    torch.cuda.synchronize()
    return s


def run(s):
    c = s.c
    if c["call"] == "sample":
        sv.sd_sample_logits_noalloc(range(s.B), s.L, s.V, s.drafts, s.q, s.logits, c["mode"], s.result, seed=s.seed)
        return s.result
    v = s.v
    if c["call"] == "load":
        for l, kv in enumerate(s.kv):
            for u in range(s.B):
                v.write_kv(u, l, 0, kv[0, s.off[u]:s.off[u + 1]], kv[1, s.off[u]:s.off[u + 1]])
        return v.kv_pool.view(torch.int16)
    if c["call"] == "draft":
        v.draft(0, s.assign, c["mode"], seed=s.seed, probs=s.probs)
        n_acc, tok = v.accept(0, s.B)
        return {"probs": s.probs, "token": tok}
    if c["call"] == "score":
        for u in range(s.B):
            v.reset_user(u, s.P[u], s.roots[u])
        v.verify(0, s.assign, s.L, s.drafts, None, "force")
        logits = v.logits(0, s.T)
        n_acc, tok = v.accept(0, s.B, commit=True)
    else:
        if s.sparse is not None:
            v.verify_sparse(0, s.assign, s.L, s.drafts, *s.sparse, c["mode"], seed=s.seed)
        else:
            v.verify(0, s.assign, s.L, s.drafts, s.q, c["mode"], seed=s.seed, stream=s.stream, graph=c["graph"])
        logits = v.logits(0, s.T, s.stream)
        n_acc, tok = v.accept(0, s.B)
        if s.stream is not None:
            torch.cuda.current_stream().wait_stream(s.stream)
    return {"logits": logits, "n_acc": n_acc, "token": tok}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    c, m = case, _model(case)
    P, L = _lengths(c)
    T, B = sum(L) + c["users"], c["users"]
    V = c.get("vocab", m.vocab)
    stop_rows = B * V * 4 if c["mode"] == "stochastic" else 0  # one draft row a user, at its stop slot
    if c["call"] == "sample":
        return {"bytes": T * V * 4 + stop_rows, "flops": 0}
    es = 2 if m.dtype == "bf16" else 4
    kv_tok = m.n_layers * 2 * m.n_kv_heads * m.head_dim * es
    if c["call"] == "load":
        return {"bytes": 2 * sum(P) * kv_tok, "flops": 0}
    nq = m.n_q_heads * m.head_dim
    per_layer = sum(a * b for a, b in (f(m) for _, f in LAYER_SHAPES))
    weights = (m.n_layers * per_layer + m.vocab * m.d_model) * es
    ctx = sum(p + l + 1 for p, l in zip(P, L))
    seen = sum((l + 1) * p + (l + 1) * (l + 2) // 2 for p, l in zip(P, L))  # (query, key) pairs
    out = T * V * 4
    if c["call"] == "draft" or c["sparse"]:
        stop_rows = 0
    return {"bytes": weights + ctx * kv_tok + out + stop_rows + T * m.d_model * es,
            "flops": 2 * T * (m.n_layers * per_layer + m.vocab * m.d_model) + 4 * m.n_layers * nq * seen}


# Products carry activations at about 16 bits and round new keys and values
# to bf16, where a last-bit difference turns into a whole bf16 step of that
# element; sums are 32-bit.  The passes are 3e-5 (short contexts, where new
# keys weigh most: 1.7e-4) away from exact(), the fp32 ones 6e-7; about four
# times the larger is stated.  Whole values are decisions on those logits:
# they differ only where two candidates are that close.
def tolerance(case):
    if case["call"] == "load":
        return "exact"
    if case["call"] == "sample":
        return {"rel": 0.0, "max": 0.0, "differ": 0.01}
    rel = 3e-6 if MODELS[case["model"]][-1] == "f32" else 7e-4
    return {"rel": rel, "max": 20 * rel, "differ": 0.01}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------

def _rms(x, gain, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * gain.double()


def _mul(x, w, rows=32768):
    return torch.cat([x @ w[i:i + rows].double().t() for i in range(0, w.shape[0], rows)], dim=-1)


def exact(case, seed):
    c, m = case, _model(case)
    if c["call"] in ("sample", "load"):
        return None  # whole numbers and copied bytes
    P, L = _lengths(c)
    nd = sum(L)
    glob = _globals(m, seed)
    if c["call"] == "draft":
        drafts = torch.zeros(0, dtype=torch.int32, device="cuda")
    elif c["call"] == "score":
        drafts = _forced(c, m, seed, nd)
    else:
        drafts = _draft_rows(c, m.vocab, nd, seed)[1]
    roots = _roots(c, m, seed)
    tok, pos, o = [], [], 0
    for u in range(c["users"]):
        tok += [torch.tensor([roots[u]], device="cuda"), drafts[o:o + L[u]].long()]
        pos += [P[u] + j for j in range(L[u] + 1)]
        o += L[u]
    x = glob["embed"][torch.cat(tok)].double()
    hd, hq, hkv = m.head_dim, m.n_q_heads, m.n_kv_heads
    ang = torch.tensor(pos, dtype=torch.float64, device="cuda")[:, None] * \
        m.rope_base ** (-2.0 * torch.arange(hd // 2, dtype=torch.float64, device="cuda") / hd)
    cos, sin = ang.cos()[:, None], ang.sin()[:, None]

    def rope(y):
        a, b = y[..., :hd // 2], y[..., hd // 2:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)

    for l in range(m.n_layers):
        w = _layer(m, seed, l)
        kv = _kv(m, seed, l, P)
        h = _rms(x, w["norm1"], m.rms_eps)
        q, k, v = (_mul(h, w[n]).view(len(pos), -1, hd) for n in ("wq", "wk", "wv"))
        if m.qk_norm:
            q, k = _rms(q, w["qnorm"], m.rms_eps), _rms(k, w["knorm"], m.rms_eps)
        q, k = rope(q), rope(k)
        k, v = k.to(_dtype(m)).double(), v.to(_dtype(m)).double()  # the cache's element type
        att, t, r = [], 0, 0
        for u in range(c["users"]):
            n = L[u] + 1
            K = torch.cat([kv[0, r:r + P[u]].double(), k[t:t + n]]).permute(1, 2, 0).contiguous()
            W = torch.cat([kv[1, r:r + P[u]].double(), v[t:t + n]]).permute(1, 0, 2).contiguous()
            Q = q[t:t + n].view(n, hkv, hq // hkv, hd).permute(1, 2, 0, 3).reshape(hkv, -1, hd)
            S = (Q @ K / math.sqrt(hd)).view(hkv, hq // hkv, n, -1)
            hide = torch.ones(n, n, dtype=torch.bool, device="cuda").triu(1)
            S[..., P[u]:].masked_fill_(hide, -math.inf)
            O = S.softmax(-1).view(hkv, -1, P[u] + n) @ W
            att.append(O.view(hkv, hq // hkv, n, hd).permute(2, 0, 1, 3).reshape(n, hq * hd))
            t += n
            r += P[u]
        x = x + _mul(torch.cat(att), w["wo"])
        h = _rms(x, w["norm2"], m.rms_eps)
        x = x + _mul(torch.nn.functional.silu(_mul(h, w["wg"])) * _mul(h, w["wu"]), w["wd"])
    z = _mul(_rms(x, glob["norm_f"], m.rms_eps), glob["lm_head"])
    if c["call"] == "draft":
        return {"probs": z.softmax(-1), "token": None}
    return {"logits": z, "n_acc": None, "token": None}
