"""The work a program has this library do, as cases that can be timed and checked.

A verification step (chain and token-tree windows, one sequence up to a
long-context batch, accepted by the slim verifier or escalated to the full one,
greedy and under the sampling rules), the prefill that precedes it, and the
pieces a routing search and a drafter call on their own: a forward over a
teacher-forced window, the routing-mask cost, the draws from a row of logits.
Sizes are those of the workload configurations, the parity tests and the
benchmark; ``draw`` spreads them over the ranges between.

``exact`` evaluates the same inputs in float64 with plain torch.  What the cache
stores is part of the inputs' contract: a bf16 model's keys and values are
rounded to bf16 where they are cached, everything else stays float64.
"""
from __future__ import annotations

import ctypes as C
import math

import numpy as np
import torch

from paper_2606_12243_amd import via
from paper_2606_12243_amd.session import Session

_EPS, _THETA = 1e-5, 10000.0
_8B_ROUTE = tuple(range(8)) + tuple(range(24, 32))

# layers, width, heads, K/V heads, head size, FFN width, vocabulary, type, slim route, temperature
_MODELS = {
    "tiny_fp32": (4, 256, 4, 4, 64, 1024, 1024, "f32", (0, 3), 1.0),
    "micro_f32": (3, 128, 2, 1, 64, 256, 500, "f32", (0, 2), 1.0),
    "micro_bf16": (3, 256, 4, 2, 64, 512, 1000, "bf16", (0, 2), 1.0),
    "small_bf16_hd128": (4, 512, 8, 2, 128, 1408, 3001, "bf16", (0, 3), 1.0),
    "1b_bf16": (16, 2048, 16, 4, 128, 5632, 32000, "bf16", tuple(range(0, 16, 2)), 28.40),
    "8b_bf16": (32, 4096, 32, 8, 128, 14336, 128256, "bf16", _8B_ROUTE, 33.98),
}
# nodes per depth of the 60-node token tree (at most 4 children each)
_TREE = (4, 12, 16, 14, 9, 5)
_GEN = 64  # tokens a sequence generates before the next request takes its place


def _step(name, model, batch, k, lo, hi, tree=False, logits=False):
    """One whole step through the native driver; every draft is accepted, so the
    sequences advance by the window (the common outcome with a good drafter)."""
    return dict(name=name, kind="step", model=model, batch=batch, k=k, ctx_lo=lo, ctx_hi=hi, tree=tree, logits=logits)


def _session(name, model, batch, k, lo, hi, rule, lag=0):
    """One step through the Python session, rolled back at the end so that it can be
    repeated.  rule "full": every draft escalates, and the full verifier also feeds
    the ``lag`` tokens its cache has not seen.  rule "sampled": the sampling rules,
    every sequence owing a draw from the slim verifier."""
    return dict(name=name, kind="session", model=model, batch=batch, k=k, ctx_lo=lo, ctx_hi=hi, rule=rule, lag=lag)


def _prefill(name, model, batch, lo, hi):
    return dict(name=name, kind="prefill", model=model, batch=batch, len_lo=lo, len_hi=hi)


def _window(name, model, batch, rows, ctx, cache):
    return dict(name=name, kind="window", model=model, batch=batch, rows=rows, ctx=ctx, cache=cache)


def listed():
    return [
        # the smallest model, one sequence: what is left is launches and the host path
        _step("step_tiny_fp32", "tiny_fp32", 1, 4, 32, 32),
        # a small model serving one user, the program keeping the logits
        _step("step_1b_chain", "1b_bf16", 1, 8, 1024, 1024, logits=True),
        # the headline workload: four sequences, eight drafts each
        _step("step_8b_chain", "8b_bf16", 4, 8, 2048, 2048),
        # one user with a token tree instead of a chain
        _step("step_8b_tree", "8b_bf16", 1, 60, 4096, 4096, tree=True),
        # long-context batched serving, ragged lengths
        _step("step_8b_long", "8b_bf16", 16, 6, 4096, 8192),
        # a step whose drafts the slim verifier is not sure of, after two that it was
        _session("escalate_8b", "8b_bf16", 4, 8, 2048, 2048, "full", lag=16),
        # sampled decoding
        _session("sampled_8b", "8b_bf16", 4, 8, 2048, 2048, "sampled"),
        # four prompts arriving together
        _prefill("prefill_8b", "8b_bf16", 4, 2047, 2047),
        # one prompt on the small model
        _prefill("prefill_1b", "1b_bf16", 1, 1023, 1023),
        # the calibration forward of a routing search (a short prompt's size too)
        _window("window_8b", "8b_bf16", 1, 256, 0, "slim"),
        # ... and the reduction of its logits to the mask's cost
        dict(name="routing_cost", kind="cost", rows=256, vocab=128256, T=1.0, alpha=0.0, beta=1.0),
        # a drafter drawing its next token for every sequence, with the distributions the rules need
        dict(name="draw_rows", kind="draw", n=16, rows=32, vocab=128256, T=1.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "session", "session", "prefill", "prefill", "window", "cost", "draw"])
    model = rng.choice(["8b_bf16", "8b_bf16", "1b_bf16", "1b_bf16", "small_bf16_hd128", "micro_bf16", "tiny_fp32",
                        "micro_f32"])
    big = model in ("8b_bf16", "1b_bf16")
    if kind in ("step", "session"):
        hi = _log_int(rng, 17, 8192 if big else 1024)
        lo = rng.choice([hi, max(16, hi // 2)])
        batch = _log_int(rng, 1, 16)
        if kind == "step" and rng.random() < 0.3:
            return dict(kind="step", model=model, batch=min(batch, 4), k=rng.randint(6, 60), ctx_lo=lo, ctx_hi=hi,
                        tree=True, logits=rng.random() < 0.3)
        k = rng.randint(1, 12)
        if kind == "step":
            return dict(kind="step", model=model, batch=batch, k=k, ctx_lo=lo, ctx_hi=hi, tree=False,
                        logits=rng.random() < 0.3)
        rule = rng.choice(["full", "sampled"])
        return dict(kind="session", model=model, batch=batch, k=k, ctx_lo=lo, ctx_hi=hi, rule=rule,
                    lag=rng.randint(0, 2) * k if rule == "full" else 0)
    if kind == "prefill":
        batch = rng.randint(1, 4)
        hi = _log_int(rng, 16, 2047 if big else 1023)
        return dict(kind="prefill", model=model, batch=batch, len_lo=rng.choice([hi, max(1, hi // 3)]), len_hi=hi)
    if kind == "window":
        ctx = rng.choice([0, _log_int(rng, 16, 2048)])
        return dict(kind="window", model=model, batch=rng.randint(1, 2), rows=_log_int(rng, 16, 512), ctx=ctx,
                    cache=rng.choice(["slim", "full"]))
    vocab = rng.choice([1000, 3001, 32000, 50257, 128256])
    if kind == "cost":
        return dict(kind="cost", rows=_log_int(rng, 1, 1024), vocab=vocab, T=rng.choice([1.0, 0.7, 2.0]),
                    alpha=rng.choice([0.0, 0.1, 0.3]), beta=rng.choice([1.0, 1.2]))
    return dict(kind="draw", n=rng.randint(1, 64), rows=64, vocab=vocab, T=rng.choice([1.0, 0.7, 8.0]))


# ------------------------------------------------------------------ inputs
class _Spec:
    def __init__(self, name):
        (self.L, self.d, self.H, self.KVH, self.hd, self.F, self.V, dt, route, self.T) = _MODELS[name]
        self.route = list(route)
        self.bf16 = dt == "bf16"
        self.dtype = torch.bfloat16 if self.bf16 else torch.float32
        self.desc = dict(n_layers=self.L, d_model=self.d, n_heads=self.H, n_kv_heads=self.KVH, head_dim=self.hd,
                         d_ffn=self.F, vocab=self.V, rms_eps=_EPS, rope_theta=_THETA, dtype=dt)

    def layer_params(self):
        return self.d * (self.H + 2 * self.KVH) * self.hd + self.H * self.hd * self.d + 3 * self.F * self.d

    def shared(self):
        """Leading layers the slim route has in common with the full model."""
        n = 0
        while n < len(self.route) and self.route[n] == n:
            n += 1
        return n


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _weights(s, seed):
    """N(0, 0.02) projections and embeddings, norm gains around 1."""
    g = _gen(seed)

    def mat(*shape):
        return torch.empty(shape, dtype=s.dtype, device="cuda").normal_(0.0, 0.02, generator=g)

    def gain():
        return (1.0 + 0.1 * torch.randn(s.d, device="cuda", generator=g)).to(s.dtype)

    w = dict(embed=mat(s.V, s.d), lm_head=mat(s.V, s.d), final_norm=gain(), attn_norm=[], w_qkv=[], w_o=[], ffn_norm=[],
             w_gate_up=[], w_down=[])
    for _ in range(s.L):
        w["attn_norm"].append(gain())
        w["ffn_norm"].append(gain())
        w["w_qkv"].append(mat((s.H + 2 * s.KVH) * s.hd, s.d))
        w["w_o"].append(mat(s.d, s.H * s.hd))
        w["w_gate_up"].append(mat(2 * s.F, s.d))
        w["w_down"].append(mat(s.d, s.F))
    return w


def _blocks(n):
    return (n + via.BLOCK - 1) // via.BLOCK


def _pool_shape(s, slots, blocks):
    return (slots, s.KVH, blocks, 2, via.BLOCK * s.hd)


def _fill_context(s, full, slim, seed):
    """Cached keys and values of the context: N(0, (0.02 sqrt d)^2), the spread of a
    projected unit-RMS row, the shared leading layers alike in both caches."""
    g = _gen(seed + (1 << 32))
    std = 0.02 * math.sqrt(s.d)
    full.normal_(0.0, std, generator=g)
    slim.normal_(0.0, std, generator=g)
    for i in range(s.shared()):
        slim[i].copy_(full[i])


def _lens(lo, hi, batch):
    """Ragged lengths of a case (its own, not the seed's: they give the outputs' shapes)."""
    return [int(v) for v in np.random.default_rng([lo, hi, batch]).integers(lo, hi + 1, size=batch)]


def _tree(rng, k):
    """k nodes: the depths' budgets in order, earlier nodes expanding first."""
    parents, frontier = [], [-1]
    for budget in _TREE:
        nxt = []
        for u in frontier:
            for _ in range(4):
                if len(nxt) < budget and len(parents) < k:
                    nxt.append(len(parents))
                    parents.append(u)
        frontier = nxt
    return parents


def _inputs(case, seed):
    """Host inputs of a model case: context lengths, committed tokens, drafts."""
    s = _Spec(case["model"])
    rng = np.random.default_rng([seed, 7])
    B = case["batch"]
    toks = lambda n: rng.integers(0, s.V, size=n).tolist()
    kind = case["kind"]
    if kind == "prefill":
        lens = _lens(case["len_lo"], case["len_hi"], B)
        return s, dict(prompts={b: toks(lens[b] + 1) for b in range(B)}, lens=lens)
    if kind == "window":
        return s, dict(ctx=[case["ctx"]] * B, rows=[toks(case["rows"]) for _ in range(B)])
    ctx = _lens(case["ctx_lo"], case["ctx_hi"], B)
    k = case["k"]
    tree = case.get("tree", False)
    steps = max(1, _GEN // (len(_TREE) if tree else k)) if kind == "step" else 1 + case["lag"] // k
    committed = {b: toks(ctx[b] + 1) for b in range(B)}
    drafts = [{b: (toks(k), _tree(rng, k) if tree else None) for b in range(B)} for _ in range(steps)]
    return s, dict(ctx=ctx, committed=committed, drafts=drafts)


class _State:
    """Model, caches and outputs of a case; the library's handles go with it."""

    def __init__(self):
        self.model = self.kv = None

    def __del__(self):
        if self.kv is not None:
            self.kv.close()
        if self.model is not None:
            self.model.close()


def _handle(st, s, ctx, grow, rows, batch, drafts, fill_seed):
    per = max(_blocks(n + grow) for n in ctx) + 1
    blocks = sum(_blocks(n + grow) + 1 for n in ctx)
    st.kv = via.KV(st.model, max_seqs=batch, max_blocks_per_seq=per, blocks_full=blocks, blocks_slim=blocks,
                   max_rows=rows, max_batch=batch, max_drafts=drafts)
    if fill_seed is not None:
        _fill_context(s, st.kv.pool_view(via.CACHE_FULL), st.kv.pool_view(via.CACHE_SLIM), fill_seed)


def _zeroed(out):
    for t in (out.row_argmax, out.row_max, out.row_sumexp, out.row_gap, out.draft_logit, out.logits):
        if t is not None:
            t.zero_()
    return out


def _attach(st):
    """The next requests take the sequences' places, with the same contexts."""
    for b, toks in st.committed.items():
        if st.step is not None:
            via.check(via.via_kv_seq_release(st.kv.h, b))
    for b, (t, tp) in st.tokens.items():
        via.check(via.via_kv_seq_reserve(st.kv.h, b, len(t) - 1))
        via.check(via.via_kv_seq_set_tokens(st.kv.h, b, tp, len(t)))
    st.step = 0


def _rows_of(draft):
    tok, parents = draft
    return len(tok) if parents is None else 1 + len({p for p in parents if p >= 0})


def prepare(case, seed):
    st = _State()
    st.case = case
    kind = case["kind"]
    if kind == "cost":
        g = _gen(seed)
        shape = (case["rows"], case["vocab"])
        st.q = torch.empty(shape, device="cuda").normal_(0.0, 1.3, generator=g)
        st.p = torch.empty(shape, device="cuda").normal_(0.0, 0.5, generator=g).add_(st.q)
        st.cost = torch.empty(case["rows"], device="cuda")
        st.stream = via.stream_ptr()
        return st
    if kind == "draw":
        g = _gen(seed)
        V, R, n = case["vocab"], case["rows"], case["n"]
        st.out = via.Out(1, R, 1, V, logits=True)
        lg = st.out.logits.view(R, V).normal_(0.0, 1.3, generator=g)
        st.out.row_max.copy_(lg.amax(1))
        st.out.row_sumexp.copy_(((lg - st.out.row_max[:, None]) / case["T"]).double().exp().sum(1))
        rng = np.random.default_rng([seed, 9])
        st.rows, st.rows_p = via._i32(rng.choice(R, size=n, replace=False))
        st.u = np.minimum(rng.random(n).astype(np.float32), np.float32(0.99999))
        st.tok = torch.zeros(n, dtype=torch.int32, device="cuda")
        st.probs = torch.empty((n, V), device="cuda")
        st.stream = via.stream_ptr()
        return st
    s, inp = _inputs(case, seed)
    B = case["batch"]
    st.model = via.Model(s.desc, _weights(s, seed), s.route)
    if kind == "prefill":
        rows = sum(inp["lens"])
        _handle(st, s, inp["lens"], 0, rows, B, 1, None)
        st.sess = Session(st.model, st.kv, via.tier_params(0.9, 0.5, s.T))
        st.prompts = inp["prompts"]
        return st
    if kind == "window":
        R = case["rows"]
        _handle(st, s, inp["ctx"], R, B * R, B, 1, seed)
        for b in range(B):
            via.check(via.via_kv_seq_reserve(st.kv.h, b, case["ctx"]))
        st.cache = via.CACHE_SLIM if case["cache"] == "slim" else via.CACHE_FULL
        st.win = via.WindowBuf(list(range(B)), inp["rows"], [[]] * B, [[]] * B, max_drafts=1)
        st.out = _zeroed(via.Out(B, R, 1, s.V, logits=True))
        st.p = via.tier_params(0.9, 0.5, s.T)
        st.stream = via.stream_ptr()
        return st
    k, tree = case["k"], case.get("tree", False)
    steps = len(inp["drafts"])
    R = max(_rows_of(d) for w in inp["drafts"] for d in w.values())
    lag = case.get("lag", 0)
    _handle(st, s, inp["ctx"], (steps + 1) * max(k, 8), B * (R + lag), B, k, seed)
    st.R, st.D = R, k
    if kind == "step":
        st.slim = _zeroed(via.Out(B, R, k, s.V, case["logits"]))
        st.full = _zeroed(via.Out(B, R, k, s.V, case["logits"]))
        st.dec = via.Dec(B, k)
        st.p = via.tier_params(0.0, 0.0, s.T)  # every confidence clears the thresholds
        st.committed = inp["committed"]
        st.tokens = {b: via._i32(t) for b, t in inp["committed"].items()}
        st.drafts = [via.DraftsBuf(w) for w in inp["drafts"]]
        st.stream = via.stream_ptr()
        st.step = None
        _attach(st)
        return st
    sampled = case["rule"] == "sampled"
    st.sess = sess = Session(st.model, st.kv, via.tier_params(0.0, 0.0, s.T), logits=True)
    for o in (sess.out_slim, sess.out_full):
        _zeroed(o)
    for b in range(B):
        sess.reserve(b, inp["committed"][b])
    for w in inp["drafts"][:-1]:  # accepted without the full verifier: its cache lags
        sess.step(w)
    st.drafts = inp["drafts"][-1]
    # thresholds no confidence, and then every confidence, reaches
    sess.p = via.tier_params(2.0, 0.0 if sampled else 2.0, s.T)
    st.sampling = None
    if sampled:
        g = _gen(seed + (2 << 32))
        z = torch.randn((B, k, s.V), generator=g, device="cuda") * 1.5
        for b in range(B):
            z[b, torch.arange(k, device="cuda"), torch.tensor(st.drafts[b][0], device="cuda")] += 4.0
        u = np.random.default_rng([seed, 8]).random((B, k, 3)).astype(np.float32)
        st.sampling = via.Sampling(0.0, 1.0, torch.softmax(z, -1), np.minimum(u, np.float32(0.99999)))
    n = np.array([len(sess.tokens[b]) for b in range(B)], np.int32)
    st.back = dict(status=np.full(B, 2, np.int32), kappa=np.zeros(B, np.int32), emit=np.full(B, -1, np.int32), new_len=n,
                   path=np.full((B, k), -1, np.int32))
    return st


# --------------------------------------------------------------------- run
def _outputs(out, dec, B, R, D, vocab):
    """What a step computes, in the entry points' layout (token ids left to the logits they come from)."""
    got = dict(row_max=out.row_max[:B * R], row_sumexp=out.row_sumexp[:B * R], row_gap=out.row_gap[:B * R])
    if D:
        got["draft_logit"] = out.draft_logit[:B * D]
    if out.logits is not None:
        got["logits"] = out.logits[:B * R * vocab]
    if dec is not None:
        got["tier"], got["conf"] = dec.tier[:B * D], dec.conf[:B * D]
    return got


def run(st):
    case = st.case
    kind = case["kind"]
    if kind == "cost":
        via.check(via.via_dimr_cost(st.q.data_ptr(), st.p.data_ptr(), case["rows"], case["vocab"], case["vocab"],
                                    case["T"], case["alpha"], case["beta"], st.cost.data_ptr(), st.stream))
        return st.cost
    if kind == "draw":
        via.check(via.via_sample_rows_static(C.byref(st.out.c), case["rows"], case["vocab"], case["n"], st.rows_p,
                                             case["T"], st.u.ctypes.data, st.tok.data_ptr(), st.probs.data_ptr(),
                                             case["vocab"], st.stream))
        return dict(tokens=st.tok, probs=st.probs)
    vocab = st.model.desc["vocab"]
    if kind == "step":
        if st.step == len(st.drafts):
            _attach(st)
        d = st.drafts[st.step]
        via.check(via.via_step(st.model.h, st.kv.h, C.byref(d.c), C.byref(st.p), C.byref(st.slim.c),
                               C.byref(st.full.c), C.byref(st.dec.c), st.stream))
        st.step += 1
        return _outputs(st.slim, st.dec, case["batch"], st.R, st.D, vocab)
    if kind == "session":
        w, h, ran = st.sess.begin(st.drafts, st.sampling)
        st.sess.commit(w, st.drafts, st.back)
        B = case["batch"]
        got = dict(slim=_outputs(st.sess.out_slim, st.sess.dec, B, st.R, st.D, vocab))
        if case["rule"] == "full":
            got["full"] = _outputs(st.sess.out_full, None, B, st.R, st.D, vocab)
        return got
    if kind == "prefill":
        st.sess.prefill_batch(st.prompts)
        for b in st.prompts:
            st.sess.release(b)
        return dict(full=st.kv.pool_full, slim=st.kv.pool_slim)
    via.check(via.via_verify_probe(st.model.h, st.kv.h, st.cache, C.byref(st.win.c), C.byref(st.p), C.byref(st.out.c),
                                   st.stream))
    return _outputs(st.out, None, case["batch"], case["rows"], 0, vocab)


# ------------------------------------------------------- work and tolerance
def _forward_work(s, layers, rows, keys_read, keys_seen, head_rows, logits):
    """Bytes and operations of one forward: weights once, cached keys and values read
    and written once, the head; keys_seen sums the keys every row attends to."""
    e = 2 if s.bf16 else 4
    kv = 2 * s.KVH * s.hd * e
    by = layers * (s.layer_params() * e + (keys_read + rows) * kv) + rows * s.d * e
    fl = layers * (2.0 * rows * s.layer_params() + 4.0 * s.H * s.hd * keys_seen)
    if head_rows:
        by += s.V * s.d * e + head_rows * 16 + (head_rows * s.V * 4 if logits else 0)
        fl += 2.0 * head_rows * s.V * s.d
    return by, fl


def work(case):
    kind = case["kind"]
    if kind == "cost":
        n = case["rows"] * case["vocab"]
        return dict(bytes=8 * n + 4 * case["rows"], flops=16 * n)
    if kind == "draw":
        n = case["n"] * case["vocab"]
        return dict(bytes=8 * n, flops=8 * n)
    s = _Spec(case["model"])
    B = case["batch"]
    if kind == "prefill":
        lens = _lens(case["len_lo"], case["len_hi"], B)
        rows, seen = sum(lens), sum(n * (n + 1) / 2 for n in lens)
        slim = len(s.route) - (s.shared() if s.shared() < len(s.route) else 0)
        f = _forward_work(s, s.L, rows, 0, seen, 0, False)
        g = _forward_work(s, slim, rows, 0, seen, 0, False)
        return dict(bytes=f[0] + g[0], flops=f[1] + g[1])
    if kind == "window":
        R, n = case["rows"], case["ctx"]
        L = len(s.route) if case["cache"] == "slim" else s.L
        by, fl = _forward_work(s, L, B * R, B * n, B * (R * n + R * (R + 1) / 2), B * R, True)
        return dict(bytes=by, flops=fl)
    n, k = sum(_lens(case["ctx_lo"], case["ctx_hi"], B)) / B, case["k"]
    R = 1 + len({p for p in _tree(None, k) if p >= 0}) if case.get("tree") else k
    logits = case.get("logits", True)
    by, fl = _forward_work(s, len(s.route), B * R, B * n, B * R * (n + R / 2), B * R, logits)
    if case.get("rule") == "full":
        r = R + case["lag"]
        f = _forward_work(s, s.L - s.shared(), B * r, B * n, B * r * (n + r / 2), B * R, True)
        by, fl = by + f[0], fl + f[1]
    return dict(bytes=by, flops=fl)


def tolerance(case):
    """About four times the error against float64 that was measured.  In a bf16 model a
    rounding difference flips the last bit of some cached keys and values, which later
    layers carry on: where the whole context is computed (prefill, window) that is most
    of the error, and the gap between two nearly equal logits shows it most."""
    kind = case["kind"]
    if kind == "cost":
        return dict(rel=2e-5)
    if kind == "draw":
        return dict(rel=1e-6, max=2e-5)
    if _MODELS[case["model"]][7] == "f32":
        return dict(rel=3e-5)
    return dict(rel={"prefill": 8e-3, "window": 3e-2}.get(kind, 5e-3))


# -------------------------------------------------------------------- exact
def _rope(x, pos, s):
    j = torch.arange(s.hd // 2, dtype=torch.float64, device=x.device)
    a = pos.double()[:, None] * torch.pow(torch.tensor(_THETA, dtype=torch.float64, device=x.device), -2.0 * j / s.hd)
    cs, sn = torch.cos(a)[:, None], torch.sin(a)[:, None]
    x1, x2 = x[..., :s.hd // 2], x[..., s.hd // 2:]
    return torch.cat([x1 * cs - x2 * sn, x2 * cs + x1 * sn], -1)


def _rms(x, g):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + _EPS) * g.double()


def _mm(x, w):
    """x w^T in float64, the weight converted a band of rows at a time."""
    return torch.cat([x @ c.double().t().contiguous() for c in w.split(16384)], -1)


def _forward(s, w, layers, tok, pos, spans, ctx_kv, masks):
    """Residual stream after ``layers`` and each layer's keys and values of the fed rows.
    spans: (first row, rows) of every sequence; ctx_kv(slot, b): cached keys and values or
    None; masks[b]: visible window rows of every window row."""
    x = w["embed"][tok].double()
    kvs = []
    G = s.H // s.KVH
    for slot, l in enumerate(layers):
        qkv = _mm(_rms(x, w["attn_norm"][l]), w["w_qkv"][l]).view(-1, s.H + 2 * s.KVH, s.hd)
        q = _rope(qkv[:, :s.H], pos, s)
        kk = _rope(qkv[:, s.H:s.H + s.KVH], pos, s).to(s.dtype).double()
        vv = qkv[:, s.H + s.KVH:].to(s.dtype).double()
        kvs.append((kk, vv))
        att = torch.empty((x.shape[0], s.H, s.hd), dtype=torch.float64, device=x.device)
        for b, (r0, n) in enumerate(spans):
            K, V = kk[r0:r0 + n], vv[r0:r0 + n]
            c = ctx_kv(slot, b)
            nc = 0
            if c is not None:
                nc = c[0].shape[0]
                K, V = torch.cat([c[0].double(), K]), torch.cat([c[1].double(), V])
            vis = torch.cat([torch.ones((n, nc), dtype=torch.bool, device=x.device), masks[b]], 1)
            for g in range(s.KVH):
                qg = q[r0:r0 + n, g * G:(g + 1) * G].reshape(n * G, s.hd)
                sc = (qg @ K[:, g].t().contiguous()).view(n, G, -1) / math.sqrt(s.hd)
                p = torch.softmax(sc.masked_fill(~vis[:, None], float("-inf")), -1)
                att[r0:r0 + n, g * G:(g + 1) * G] = (p.reshape(n * G, -1) @ V[:, g].contiguous()).view(n, G, s.hd)
        x = x + _mm(att.reshape(-1, s.H * s.hd), w["w_o"][l])
        gu = _mm(_rms(x, w["ffn_norm"][l]), w["w_gate_up"][l])
        x = x + _mm(torch.nn.functional.silu(gu[:, :s.F]) * gu[:, s.F:], w["w_down"][l])
    return x, kvs


def _paged(pool, s, first, n):
    """slot -> keys and values [n, KVH, hd] of a sequence whose pages start at block ``first``."""
    def get(slot):
        nb = _blocks(n)
        pg = pool[slot, :, first:first + nb]
        K = pg[:, :, 0].reshape(s.KVH, nb, s.hd // 8, via.BLOCK, 8).permute(1, 3, 0, 2, 4).reshape(-1, s.KVH, s.hd)
        V = pg[:, :, 1].reshape(s.KVH, nb, s.hd, via.BLOCK).permute(1, 3, 0, 2).reshape(-1, s.KVH, s.hd)
        return K[:n], V[:n]
    return get


def _page_out(pool, s, slot, first, K, V):
    n, nb = K.shape[0], _blocks(K.shape[0])
    pad = torch.zeros((nb * via.BLOCK - n, s.KVH, s.hd), dtype=K.dtype, device=K.device)
    K, V = torch.cat([K, pad]), torch.cat([V, pad])
    pool[slot, :, first:first + nb, 0] = K.view(nb, via.BLOCK, s.KVH, s.hd // 8, 8).permute(2, 0, 3, 1, 4).reshape(
        s.KVH, nb, -1)
    pool[slot, :, first:first + nb, 1] = V.view(nb, via.BLOCK, s.KVH, s.hd).permute(2, 0, 3, 1).reshape(s.KVH, nb, -1)


def _stats(lg, T, logits):
    """Row statistics of float64 logits in the entry points' layout."""
    top = lg.topk(2, -1).values
    got = dict(row_max=top[:, 0], row_sumexp=torch.exp((lg - top[:, :1]) / T).sum(-1), row_gap=top[:, 0] - top[:, 1])
    if logits:
        got["logits"] = lg.reshape(-1)
    return got


def exact(case, seed):
    kind = case["kind"]
    if kind == "cost":
        st = prepare(case, seed)
        rows = []
        for r in range(case["rows"]):
            lq = torch.log_softmax(st.q[r].double() / case["T"], -1)
            lp = torch.log_softmax(st.p[r].double() / case["T"], -1)
            a = torch.relu(math.log(1 - case["alpha"]) + lp - lq)
            b = torch.relu(math.log(case["beta"]) + lp - lq)
            rows.append((lp.exp() * a).sum() + (lq.exp() * b).sum())
        return torch.stack(rows)
    if kind == "draw":
        st = prepare(case, seed)
        lg = st.out.logits.view(case["rows"], -1)[torch.as_tensor(st.rows, dtype=torch.long, device="cuda")]
        return dict(tokens=None, probs=torch.softmax(lg.double() / case["T"], -1))
    s, inp = _inputs(case, seed)
    B = case["batch"]
    w = _weights(s, seed)
    causal = lambda n: torch.ones((n, n), dtype=torch.bool, device="cuda").tril()
    if kind == "prefill":
        lens = inp["lens"]
        starts = np.concatenate([[0], np.cumsum(lens)]).tolist()
        first = np.concatenate([[0], np.cumsum([_blocks(n) for n in lens])]).tolist()
        tok = torch.tensor([t for b in range(B) for t in inp["prompts"][b][:-1]], device="cuda")
        pos = torch.cat([torch.arange(n, device="cuda") for n in lens])
        spans = [(starts[b], lens[b]) for b in range(B)]
        blocks = sum(_blocks(n) + 1 for n in lens)
        got = {}
        for name, layers in (("full", list(range(s.L))), ("slim", s.route)):
            pool = torch.zeros(_pool_shape(s, len(layers), blocks), dtype=torch.float64, device="cuda")
            _, kvs = _forward(s, w, layers, tok, pos, spans, lambda slot, b: None, [causal(n) for n in lens])
            for slot, (K, V) in enumerate(kvs):
                for b, (r0, n) in enumerate(spans):
                    _page_out(pool, s, slot, first[b], K[r0:r0 + n], V[r0:r0 + n])
            got[name] = pool.reshape(-1)
        return got
    ctx = inp["ctx"]
    # the tokens each sequence feeds past its context, their depths and what they see of each other
    feed, depth, masks, head = [], [], [], []
    k, tree = case.get("k", 0), case.get("tree", False)
    if kind == "window":
        grow, R = case["rows"], case["rows"]
        for b in range(B):
            feed.append(inp["rows"][b])
            depth.append(list(range(R)))
            masks.append(causal(R))
            head.append(list(range(R)))
    else:
        grow = (len(inp["drafts"]) + 1) * max(k, 8)
        R = max(_rows_of(d) for wd in inp["drafts"] for d in wd.values())
        wins = inp["drafts"][:1] if kind == "step" else inp["drafts"]
        for b in range(B):
            toks = [inp["committed"][b][-1]]
            if tree:
                dt, par = wins[0][b]
                rn = [-1] + sorted({p for p in par if p >= 0})
                dep = {-1: 0}
                for j, p in enumerate(par):
                    dep[j] = dep[p] + 1
                toks += [dt[u] for u in rn[1:]]
                m = torch.zeros((len(rn), len(rn)), dtype=torch.bool)
                for r, u in enumerate(rn):
                    while u >= 0:
                        m[r, rn.index(u)] = True
                        u = par[u]
                    m[r, 0] = True
                masks.append(m.cuda())
                depth.append([dep[u] for u in rn])
            else:
                for wd in wins:
                    toks += wd[b][0]
                toks = toks[:-1]
                masks.append(causal(len(toks)))
                depth.append(list(range(len(toks))))
            feed.append(toks)
            head.append(list(range(len(toks) - R, len(toks))))
    blocks = sum(_blocks(n + grow) + 1 for n in ctx)
    pools = [torch.zeros(_pool_shape(s, n, blocks), dtype=s.dtype, device="cuda") for n in (s.L, len(s.route))]
    _fill_context(s, pools[0], pools[1], seed)
    first = np.concatenate([[0], np.cumsum([_blocks(n) for n in ctx])]).tolist()
    starts = np.concatenate([[0], np.cumsum([len(f) for f in feed])]).tolist()
    spans = [(starts[b], len(feed[b])) for b in range(B)]
    tok = torch.tensor([t for f in feed for t in f], device="cuda")
    pos = torch.tensor([ctx[b] + d for b in range(B) for d in depth[b]], device="cuda")
    rows = torch.tensor([starts[b] + r for b in range(B) for r in head[b]], device="cuda")

    def logits_of(cache):
        layers = s.route if cache == via.CACHE_SLIM else list(range(s.L))
        get = [_paged(pools[cache], s, first[b], ctx[b]) for b in range(B)]
        x, _ = _forward(s, w, layers, tok, pos, spans, lambda slot, b: get[b](slot) if ctx[b] else None, masks)
        return _mm(_rms(x[rows], w["final_norm"]), w["lm_head"])

    def outputs(lg, with_logits, with_dec):
        got = _stats(lg, s.T, with_logits)
        if k == 0:
            return got
        at = []
        for b in range(B):
            dt, par = wins[-1][b]
            row_of = {u: r for r, u in enumerate([-1] + sorted({p for p in par if p >= 0}))} if tree else None
            at += [(b * R + (row_of[par[j]] if tree else j), dt[j]) for j in range(k)]
        r = torch.tensor([a[0] for a in at], device="cuda")
        dl = lg[r, torch.tensor([a[1] for a in at], device="cuda")]
        got["draft_logit"] = dl
        if with_dec:
            got["tier"] = None
            got["conf"] = torch.exp((dl - got["row_max"][r]) / s.T)
        return got

    if kind == "window":
        return outputs(logits_of(via.CACHE_SLIM if case["cache"] == "slim" else via.CACHE_FULL), True, False)
    if kind == "step":
        return outputs(logits_of(via.CACHE_SLIM), case["logits"], True)
    got = dict(slim=outputs(logits_of(via.CACHE_SLIM), True, True))
    if case["rule"] == "full":
        got["full"] = outputs(logits_of(via.CACHE_FULL), True, False)
    return got
