"""The calls a serving program makes of this framework, as measurable cases.

Three kinds:
  decode   attention of one step over a resident mixed bf16 / int4 history,
           once per layer (the step's token was appended by its own call, or a
           speculative query is scored without being kept);
  serve    requests from an empty cache: reset, bulk append of the prompts
           (kept HIGH, or labelled and governed by the table), bulk append of
           tokens generated earlier (a request resumed after preemption), then
           decode steps that persist their token and attend the history;
  distort  the calibration measure of Eq. 4 over two resident caches.

The reference in exact() is plain torch in float64: the table's rule, the
online controller, the int4 format and the attention, by their definitions.
"""

from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2608_28276_amd import pask
from paper_2608_28276_amd.session import PaskSession
from workload.policy import make_policy, pack_blob, with_budget_controller
from workload.tags import CRITICAL_STATES, PARSER_STATES, function_call_tags_with_states, schema_prompt_tags, tag_mix

DROP, LOW, HIGH = 0, 1, 2
BUCKET_TAG = 2                       # arg_value: the bucket of the distortion cases
_BASE = dict(kind="decode", batch=1, layers=1, hq=32, hkv=8, dim=128, pmin=1024, pmax=1024, tagged=False, sink=0,
             beta=0.33, history=0, steps=0, window=0, states=False, noalloc=False, action=LOW)


def _case(name=None, **kw):
    c = dict(_BASE, **kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest calls: one short sequence, two layers of a small model, under code that may not allocate.
        _case("decode_tiny_b1", layers=2, hq=8, hkv=2, dim=64, pmin=256, pmax=256, history=128, noalloc=True),
        # One user: a 2k prompt and the first 16 tokens of the answer, four layers.
        _case("request_b1", kind="serve", layers=4, pmin=2048, pmax=2048, steps=16),
        # A handful of sequences (48 sequence-head segments), ragged prompts.
        _case("decode_b6", batch=6, layers=4, pmin=1024, pmax=8192, history=512),
        # The serving batch of the benchmark, prompts kept HIGH.
        _case("decode_b64", batch=64, layers=2, pmin=1024, pmax=8192, history=512),
        # Prompt-side tables make most of the history int4; a model with 8 query heads per KV head.
        _case("decode_tagged_g8_b128", batch=128, hq=64, pmin=4096, pmax=16384, tagged=True, sink=16, history=256),
        # Many short chats at once: more sequences than one wave holds, eight steps.
        _case("chat_b384", kind="serve", batch=384, pmin=64, pmax=768, steps=8),
        # Prefill of the serving batch, prompts kept HIGH, and the first step.
        _case("prompt_b64", kind="serve", batch=64, pmin=1024, pmax=8192, steps=1),
        # Prefill of one long labelled prompt, as requests arrive one by one, and the first step.
        _case("prompt_tagged_b1_32k", kind="serve", layers=2, pmin=32000, pmax=32000, tagged=True, sink=16, steps=1),
        # Prefill of a batch of labelled prompts (most tokens int4 or released), and the first step.
        _case("prompt_tagged_b32", kind="serve", batch=32, pmin=4096, pmax=16384, tagged=True, sink=16, steps=1),
        # The protected recent window: prompts, then 16 steps in which tokens leave the window.
        _case("window_b64", kind="serve", batch=64, pmin=512, pmax=2048, window=64, steps=16),
        # The online controller: requests resumed with 384 generated tokens replayed, then eight steps.
        _case("resume_controller_b16", kind="serve", batch=16, layers=2, pmin=512, pmax=2048, states=True,
              history=384, steps=8),
        # Calibration: reference against an intervention that releases one bucket, two layers.
        _case("distortion_b16", kind="distort", batch=16, layers=2, pmin=1024, pmax=4096, history=512, action=DROP),
    ]


_HEADS = [(8, 2), (32, 8), (64, 8), (16, 8), (8, 8), (4, 1), (6, 3), (40, 5), (28, 7), (16, 4)]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    most = max(work(c)["bytes"] for c in listed())
    while True:
        kind = rng.choice(["decode", "decode", "serve", "serve", "serve", "distort"])
        hq, hkv = rng.choice(_HEADS)
        pmax = _log_int(rng, 33, 32768)
        c = _case(kind=kind, hq=hq, hkv=hkv, dim=rng.choice([64, 128, 128]), batch=_log_int(rng, 1, 400),
                  layers=rng.choice([1, 2, 4]), pmin=max(17, int(pmax * rng.uniform(0.1, 1.0))), pmax=pmax,
                  beta=rng.choice([0.25, 0.33, 0.5, 1.0]), history=_log_int(rng, 1, 1024), noalloc=False)
        if kind == "serve":
            c["steps"] = rng.randint(1, 16)
            c["tagged"] = rng.random() < 0.4
            c["history"] = rng.choice([0, rng.randint(1, 400)])
            style = rng.random()
            if style < 0.2 and not c["tagged"]:
                c["states"] = True
            elif style < 0.4:
                c["window"] = rng.randint(5, 130)
        elif kind == "decode":
            c["tagged"] = rng.random() < 0.4
            c["noalloc"] = rng.random() < 0.2
        else:
            c["action"] = rng.choice([DROP, LOW])
        if c["tagged"]:
            c["sink"] = 16
        if 1e5 < work(c)["bytes"] <= most and 2 * c["batch"] * c["pmax"] * c["hkv"] * c["dim"] * 2 < 10e9:
            return c


# ---- host-side inputs: tag streams, the frozen table, prompt lengths -------------------------------------------------
@functools.lru_cache(None)
def _generated_stream():
    return function_call_tags_with_states(8192, 71)


@functools.lru_cache(None)
def _prompt_stream():
    return schema_prompt_tags(65536, 72)


@functools.lru_cache(None)
def _policy(tagged, layers, beta, sink, window, states):
    gen, st = _generated_stream()
    mix = tag_mix(np.concatenate([_prompt_stream(), gen]), 12) if tagged else tag_mix(gen, 6)
    pol = make_policy(12 if tagged else 6, layers, layers, beta, 1002, tag_probs=mix, n_sink=sink)
    if states:
        pol = with_budget_controller(pol, [(gen[i:i + 512], st[i:i + 512]) for i in range(0, 4096, 512)],
                                     len(PARSER_STATES), CRITICAL_STATES)
    pol.recent_window = window
    return pol


def _policy_of(c):
    return _policy(c["tagged"], c["layers"], c["beta"], c["sink"], c["window"], c["states"])


def _intervened(pol, action):
    """(reference, intervention): every bucket HIGH, and bucket (arg_value, every group) given `action`."""
    from dataclasses import replace
    full = np.full_like(np.asarray(pol.action), HIGH)
    itv = full.copy()
    itv[BUCKET_TAG] = action
    zero = np.zeros_like(full)
    return replace(pol, action=full, floor=zero), replace(pol, action=itv, floor=zero)


def _host(c, seed):
    """Prompt lengths (spread evenly over the range, in random order) and tag streams of every sequence."""
    rng = np.random.default_rng([seed, 11])
    B, T = c["batch"], c["history"] + c["steps"]
    u = (rng.permutation(B) + rng.uniform(0, 1, B)) / B
    lens = np.minimum(c["pmax"], c["pmin"] + np.floor(u * (c["pmax"] - c["pmin"] + 1))).astype(np.int32)
    gen, st = _generated_stream()
    at = rng.integers(0, gen.size - T, B)
    gtags = np.stack([gen[a:a + T] for a in at]) if T else np.zeros((B, 0), np.uint8)
    states = np.stack([st[a:a + T] for a in at]) if T else np.zeros((B, 0), np.uint8)
    ptags = None
    if c["tagged"]:
        p = _prompt_stream()
        at = rng.integers(0, p.size - c["pmax"], B)
        ptags = np.stack([p[a:a + c["pmax"]] for a in at])
    return lens, ptags, gtags, states


# ---- device inputs ---------------------------------------------------------------------------------------------------
def _randn(shape, seed, purpose, layer):
    g = torch.Generator(device="cuda")
    g.manual_seed((seed * 1009 + purpose) * 131 + layer)
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)


def _kv(c, seed, purpose, layer, rows):
    """bf16 K and V [batch, rows, hkv, dim]; K with a few channels four times as wide, as trained keys have."""
    shape = (c["batch"], rows, c["hkv"], c["dim"])
    k, v = _randn(shape, seed, purpose, layer), _randn(shape, seed, purpose + 1, layer)
    k[..., 3::37] *= 4
    return k, v


def _queries(c, seed):
    return _randn((max(1, c["steps"]), c["layers"], c["batch"], c["hq"], c["dim"]), seed, 9, 0)


def _session(c, pol, lens):
    longest = c["pmax"] + c["history"] + c["steps"]
    pages = c["layers"] * (int(np.sum((lens + c["history"] + c["steps"] + 15) // 16)) + c["batch"])
    return PaskSession(pack_blob(pol), max_batch=c["batch"], n_layers=c["layers"], n_q_heads=c["hq"],
                       n_kv_heads=c["hkv"], head_dim=c["dim"], max_tokens_per_seq=longest, hi_pages=pages,
                       lo_pages=pages, max_ctx_hint=longest, prefill=0)


def prepare(case, seed):
    c = case
    lens, ptags, gtags, states = _host(c, seed)
    dev = lambda x: None if x is None else torch.as_tensor(np.ascontiguousarray(x), device="cuda")
    s = dict(case=c, n_new=dev(lens), ptags=dev(ptags), q=_queries(c, seed))
    h = c["history"]
    shape = (max(1, c["steps"]), c["layers"], c["batch"], c["hq"])
    s["out"] = torch.zeros(shape + (c["dim"],), dtype=torch.bfloat16, device="cuda")
    s["lse"] = torch.zeros(shape, dtype=torch.float32, device="cuda")
    s["htags"] = dev(gtags[:, :h]) if h else None
    s["hstates"] = dev(states[:, :h]) if h and c["states"] else None
    if c["kind"] == "serve":
        s["sess"] = _session(c, _policy_of(c), lens)
        s["prompt"] = [_kv(c, seed, 1, l, c["pmax"]) for l in range(c["layers"])]
        s["hist"] = [_kv(c, seed, 3, l, h) for l in range(c["layers"])] if h else None
        s["new"] = [[tuple(x[:, 0].contiguous() for x in _kv(c, seed, 20 + 2 * t, l, 1)) for l in range(c["layers"])]
                    for t in range(c["steps"])]
        s["tags"] = [dev(gtags[:, h + t]) for t in range(c["steps"])]
        s["states"] = [dev(states[:, h + t]) if c["states"] else None for t in range(c["steps"])]
        return s
    pols = [_policy_of(c)] if c["kind"] == "decode" else _intervened(_policy_of(c), c["action"])
    s["sessions"] = [_session(c, p, lens) for p in pols]
    for l in range(c["layers"]):
        k, v = _kv(c, seed, 1, l, c["pmax"])
        hk, hv = _kv(c, seed, 3, l, h) if h else (None, None)
        for sess in s["sessions"]:
            sess.append(l, s["ptags"], k, v, n_new=s["n_new"], keep_all=not c["tagged"])
            if h:
                sess.append(l, s["htags"], hk, hv)
        del k, v, hk, hv
    if c["kind"] == "distort":
        a = s["sessions"][0]
        s["in_s"] = dev((gtags == BUCKET_TAG).any(1).astype(np.uint8))
        s["ws"] = torch.empty(2 * a.ws_bytes, dtype=torch.uint8, device="cuda")
        s["dist"] = torch.zeros(c["batch"], dtype=torch.float32, device="cuda")
    torch.cuda.empty_cache()
    return s


def run(s):
    c = s["case"]
    if c["kind"] == "decode":
        sess = s["sessions"][0]
        step = sess.decode_noalloc if c["noalloc"] else sess.decode
        for l in range(c["layers"]):
            step(l, s["q"][0, l], s["out"][0, l], s["lse"][0, l])
        return {"out": s["out"], "lse": s["lse"]}
    if c["kind"] == "distort":
        a, b = s["sessions"]
        s["dist"].zero_()
        for l in range(c["layers"]):
            pask.pask_attn_distortion(a.cache, b.cache, l, c["batch"], s["q"][0, l], s["in_s"], a.softmax_scale,
                                      a.max_ctx_hint, s["ws"], 2 * a.ws_bytes, s["dist"], a.stream)
        return {"dist": s["dist"]}
    sess = s["sess"]
    sess.reset()
    if c["states"]:
        sess.budget_init(c["history"] + c["steps"])
    for l in range(c["layers"]):
        k, v = s["prompt"][l]
        sess.append(l, s["ptags"], k, v, n_new=s["n_new"], keep_all=not c["tagged"])
        if s["hist"]:
            k, v = s["hist"][l]
            sess.append(l, s["htags"], k, v, states=s["hstates"])
    for t in range(c["steps"]):
        for l in range(c["layers"]):
            k, v = s["new"][t][l]
            sess.decode(l, s["q"][t, l], s["out"][t, l], s["lse"][t, l], s["tags"][t], k, v,
                        states_new=s["states"][t])
    res = {"out": s["out"], "lse": s["lse"], "counters": sess.counters(), "lists": sess.index_lists()}
    if c["batch"] == 1:                  # one sequence: its pages are granted in order, so the stores compare as bytes
        res["hi"], res["lo"] = sess.hi_pool(), sess.lo_pool()
    return res


# ---- the bytes and operations a pass cannot do without ---------------------------------------------------------------
@functools.lru_cache(None)
def _shares(tagged, layers, beta, sink, which, kind, action):
    """(HIGH, LOW) share of the table-governed tokens, mean over the layers."""
    pol = _policy(tagged, layers, beta, sink, 0, False)
    if kind == "distort":
        ref, itv = _intervened(pol, action)
        gen = _generated_stream()[0]
        return [(np.mean([np.mean(p.action[gen, g] == a) for g in range(layers)])) for p in (ref, itv)
                for a in (HIGH, LOW)]
    z = _prompt_stream() if which == "prompt" else _generated_stream()[0]
    act = np.maximum(pol.action, pol.floor)[z]
    return float(np.mean(act == HIGH)), float(np.mean(act == LOW))


def work(case):
    c = case
    B, L, Hq, H, D = c["batch"], c["layers"], c["hq"], c["hkv"], c["dim"]
    mh, ml = 4 * H * D, 2 * H * (D // 2 + D // 16)
    P = (c["pmin"] + c["pmax"]) / 2.0
    key = (c["tagged"], L, c["beta"], c["sink"])
    ph, pl = _shares(*key, "prompt", "", 0) if c["tagged"] else (1.0, 0.0)
    qo = 4 * B * Hq * D + 4 * B * Hq
    if c["kind"] == "distort":
        rh, rl, ih, il = _shares(*key, "gen", "distort", c["action"])
        n = [P + c["history"] * h for h in (rh, ih)]
        lo = [c["history"] * x for x in (rl, il)]
        return {"bytes": L * B * (sum(n) * mh + sum(lo) * ml) + L * 2 * B * Hq * D + 4 * B,
                "flops": L * B * (sum(n) + sum(lo)) * 4.0 * Hq * D}
    gh, gl = _shares(*key, "gen", "", 0)
    hist = lambda g: (P * ph + g * gh, P * pl + g * gl)       # HIGH and LOW entries after g generated tokens
    if c["kind"] == "decode":
        nh, nl = hist(c["history"])
        return {"bytes": L * (B * (nh * mh + nl * ml) + qo), "flops": L * B * (nh + nl) * 4.0 * Hq * D}
    # appended tokens: persisted ones' rows read, their stored forms and list entries written, tags read
    g = c["history"] + c["steps"]
    nh, nl = hist(g)
    total = L * B * (nh * (2 * mh + 4) + nl * (mh + ml + 4) + g + (P if c["tagged"] else 0))
    flops = 0.0
    for t in range(c["steps"]):
        nh, nl = hist(c["history"] + t + 1)
        total += L * (B * (nh * mh + nl * ml) + qo)
        flops += L * B * (nh + nl) * 4.0 * Hq * D
    return {"bytes": total, "flops": flops}


def tolerance(case):
    # Measured against exact(), times four: outputs rounded to bf16 differ by 1.7e-3; the distortion is float32 all
    # through (2e-6 for a released bucket), but an int4 one's weights are rounded to fp16 (2e-4 on short histories).
    if case["kind"] == "distort":
        return {"rel": 1e-5 if case["action"] == DROP else 1e-3}
    return {"rel": 8e-3}


# ---- the reference, in float64 ---------------------------------------------------------------------------------------
def _dequantised(x):
    """x (bf16 [n, H, D]) as RETAIN-LOW stores it: int4, one fp16 scale per 32 elements."""
    n, H, D = x.shape
    g = x.double().view(n, H, D // 32, 32)
    s = (g.abs().amax(-1, keepdim=True) / 7.0).clamp(max=65504.0).half().double()
    q = torch.where(s > 0, torch.round(g / s.clamp(min=1e-30)), torch.zeros_like(g)).clamp(-7, 7)
    return (q * s).view(n, H, D)


def _attend(q, k, v, scale):
    """q [Hq, D], k / v [n, H, D] in float64: outputs [Hq, D] and log-sum-exps [Hq]."""
    Hq, D = q.shape
    H = k.shape[1]
    s = torch.matmul(q.view(H, Hq // H, D), k.permute(1, 2, 0).contiguous()) * scale
    o = torch.matmul(torch.softmax(s, -1), v.permute(1, 0, 2).contiguous())
    return o.reshape(Hq, D), torch.logsumexp(s, -1).reshape(Hq)


def _controlled(c, pol, tags, states):
    """Alg. 2 over one sequence's generated tokens: actions [tokens, groups]."""
    C = pol.n_groups
    mh, ml = 4 * c["hkv"] * c["dim"], 2 * c["hkv"] * (c["dim"] // 2 + c["dim"] // 16)
    m = [0, ml, mh]                                   # one layer per group
    R = int(pol.beta_q) * len(tags) * C * mh // 65536
    gamma = [int(r) * C * mh // 16 for r in pol.reserve_q]
    a0 = np.maximum(pol.action, pol.floor).astype(int).tolist()
    floor, rho = pol.floor.astype(int).tolist(), pol.rho_up.tolist()
    res = np.zeros((len(tags), C), np.int64)
    for i, (z, s) in enumerate(zip(tags.tolist(), states.tolist())):
        a = list(a0[z])
        cost = sum(m[x] for x in a)
        B = max(0, R - gamma[s])
        while cost > B:
            can = [g for g in range(C) if a[g] > floor[z][g]]
            if not can:
                break
            g = min(can, key=lambda g: (rho[z][g][a[g] - 1], g))
            cost -= m[a[g]] - m[a[g] - 1]
            a[g] -= 1
        while pol.crit[s]:
            can = [g for g in range(C) if a[g] < HIGH and rho[z][g][a[g]] > 0 and cost + m[a[g] + 1] - m[a[g]] <= B]
            if not can:
                break
            g = max(can, key=lambda g: (rho[z][g][a[g]], -g))
            cost += m[a[g] + 1] - m[a[g]]
            a[g] += 1
        R -= cost
        res[i] = a
    return res


def _actions(c, pol, n, ptags, gtags, states, layer):
    """Action of every position of one sequence (n prompt tokens, then the generated ones) in `layer`."""
    table = np.maximum(pol.action, pol.floor)[:, layer].astype(np.int64)
    prompt = table[ptags[:n]] if ptags is not None else np.full(n, HIGH)
    gen = _controlled(c, pol, gtags, states)[:, layer] if c["states"] else table[gtags]
    act = np.concatenate([prompt, gen])
    act[:c["sink"]] = HIGH
    return act


def _stores(act, k, v):
    """Float64 K and V of a sequence as its stores hold them (released entries among them, unchanged)."""
    low = torch.as_tensor(act == LOW, device="cuda")[:, None, None]
    return torch.where(low, _dequantised(k), k.double()), torch.where(low, _dequantised(v), v.double())


def exact(case, seed):
    c = case
    lens, ptags, gtags, states = _host(c, seed)
    q = _queries(c, seed).double()
    scale = float(torch.tensor(1.0 / math.sqrt(c["dim"]), dtype=torch.float32))
    out = torch.zeros(q.shape, dtype=torch.float64, device="cuda")
    lse = torch.zeros(q.shape[:-1], dtype=torch.float64, device="cuda")
    dist = torch.zeros(c["batch"], dtype=torch.float64, device="cuda")
    pols = [_policy_of(c)] if c["kind"] != "distort" else _intervened(_policy_of(c), c["action"])
    for l in range(c["layers"]):
        rows = [_kv(c, seed, 1, l, c["pmax"])]
        if c["history"]:
            rows.append(_kv(c, seed, 3, l, c["history"]))
        rows += [_kv(c, seed, 20 + 2 * t, l, 1) for t in range(c["steps"])]
        for b in range(c["batch"]):
            n = int(lens[b])
            kb, vb = (torch.cat([rows[0][i][b, :n]] + [r[i][b] for r in rows[1:]]) for i in (0, 1))
            got = []
            for pol in pols:
                act = _actions(c, pol, n, None if ptags is None else ptags[b], gtags[b], states[b], l)
                ks, vs = _stores(act, kb, vb)
                for t in range(q.shape[0]):
                    end = n + c["history"] + (t + 1 if c["steps"] else 0)
                    old = max(0, end - c["window"])          # positions from here on are in the window
                    kept = torch.as_tensor(np.flatnonzero(act[:old] != DROP), device="cuda")
                    kk = torch.cat([ks[kept], kb[old:end].double()])
                    vv = torch.cat([vs[kept], vb[old:end].double()])
                    out[t, l, b], lse[t, l, b] = _attend(q[t, l, b], kk, vv, scale)
                got.append(out[0, l, b].clone())
            if c["kind"] == "distort" and (gtags[b] == BUCKET_TAG).any():
                dist[b] += (got[0] - got[1]).square().sum(-1).max()
        del rows
    if c["kind"] == "distort":
        return {"dist": dist}
    if c["kind"] == "decode":
        return {"out": out, "lse": lse}
    res = {"out": out, "lse": lse, "counters": None, "lists": None}
    if c["batch"] == 1:
        res["hi"] = res["lo"] = None
    return res
