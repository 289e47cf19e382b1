"""The workloads this library's performance is tracked on.

Every case is one pass through the public entry points of `paper_2604_17701_amd.binding`, as a verification server
calls them: rounds with host or device buffers, the two-call selective-hidden protocol, the speculative-sampling
round and its rule alone, and prompt ingestion.  Sizes follow `wisv_inputs.configs`: the tiny fp32 decoder, the
8B-shaped bf16 decoder, and a four-layer slice of the latter (same widths, vocabulary 32000) that keeps the balance
between layers and LM head roughly while its rounding errors stay those of a few layers.

`listed()` names the cases, `draw()` samples more from the same ranges, `prepare()` builds what a server holds before
the call, `run()` is one pass, `work()` what the pass cannot do without, `exact()` the same results in 64 bits.
"""
from __future__ import annotations

import itertools
import math
from dataclasses import replace

import numpy as np
import torch

from paper_2604_17701_amd import binding
from wisv_inputs.configs import LLAMA8B, PROTO_FH, PROTO_SH, TINY

DEV = "cuda:0"
SLICE = replace(LLAMA8B, n_layers=4, vocab=32000)      # four layers of the 8B shape
SLICE_V = replace(LLAMA8B, n_layers=4)                 # the same with the full vocabulary
MODELS = {"tiny": TINY, "full": LLAMA8B, "slice": SLICE, "slice_v": SLICE_V}


# ------------------------------------------------------------------------------------------------ the cases

def _round(name, model, batch, k, ctx, ragged, proto, call):
    """kind "round": `ctx` cached tokens per stream (ragged: between ctx / 8 and ctx), proto "fh" | "sh" | "mixed";
    call "device" (buffers on the GPU, enqueue only), "host" (host buffers), "two" (VERIFY_ONLY, then DECIDE_ONLY with
    the rows the first call asked for) or "logits" (device buffers, and the logits read back)."""
    return {"name": name, "kind": "round", "model": model, "batch": batch, "k": k, "ctx": ctx, "ragged": ragged,
            "proto": proto, "call": call}


def listed():
    return [
        # the smallest use: a toy fp32 target, host buffers, logits looked at (launches and copies are all there is)
        _round("tiny_f32_b1_k4", "tiny", 1, 4, 128, False, "fh", "host_logits"),
        # the headline workload, whole depth: one device, short context, four drafted tokens, full-hidden upload
        _round("full_b1_k4_l512", "full", 1, 4, 512, False, "fh", "logits"),
        # one device with a long context under the selective-hidden protocol as its two messages, host buffers
        _round("slice_b1_k8_l4096_two", "slice", 1, 8, 4096, False, "sh", "two"),
        # a few devices of unequal progress, odd block length: 15 rows
        _round("slice_b3_k5_ragged", "slice", 3, 5, 700, True, "mixed", "device"),
        # a small server: 32 rows
        _round("slice_b8_k4_l1024", "slice", 8, 4, 1024, False, "fh", "device"),
        # a busy server: 96 rows
        _round("slice_b16_k6_l2048", "slice", 16, 6, 2048, False, "fh", "device"),
        # odd counts all over: 143 rows, unequal contexts
        _round("slice_b13_k11_ragged", "slice", 13, 11, 3000, True, "mixed", "device"),
        # the largest: 64 devices with long contexts, both upload protocols: 512 rows
        _round("slice_b64_k8_l8192", "slice", 64, 8, 8192, False, "mixed", "device"),
        # prompt ingestion on a single-device context, and on one that serves 16 devices (odd length)
        {"name": "prefill_512_b1_k4", "kind": "prefill", "model": "slice", "batch": 1, "k": 4, "n": 512},
        {"name": "prefill_1999_b16_k6", "kind": "prefill", "model": "slice", "batch": 16, "k": 6, "n": 1999},
        # the stochastic verifier: its rule alone on a large batch, and a whole round of it (28 rows)
        {"name": "ss_rule_b64_k8", "kind": "ss_rule", "batch": 64, "k": 8, "vocab": 128256},
        {"name": "ss_round_b4_k7_l900", "kind": "ss_round", "model": "slice_v", "batch": 4, "k": 7, "ctx": 900},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["round", "round", "round", "round", "prefill", "ss_rule", "ss_round"])
    if kind == "ss_rule":
        k = rng.randint(1, 16)
        return {"kind": kind, "batch": min(_log(rng, 1, 64), 512 // k), "k": k, "vocab": _log(rng, 997, 128256)}
    if kind == "prefill":
        k = rng.randint(1, 16)
        return {"kind": kind, "model": "slice", "batch": min(_log(rng, 1, 16), 256 // k), "k": k,
                "n": min(_log(rng, 24, 1999), 192 * k)}
    k = rng.randint(1, 16)
    if kind == "ss_round":
        return {"kind": kind, "model": "slice_v", "batch": min(_log(rng, 1, 24), 160 // k), "k": k, "ctx": _log(rng, 40, 3000)}
    batch = min(_log(rng, 1, 64), 512 // k)
    if rng.random() < 0.1:
        c = _round("", "tiny", 1, k, _log(rng, 16, 1000), False, "fh", "host_logits")
        del c["name"]
        return c
    c = _round("", "slice", batch, k, _log(rng, 40, 8192), rng.random() < 0.5, rng.choice(["fh", "sh", "mixed"]),
               rng.choice(["device", "device", "device", "host", "two"]))
    del c["name"]
    return c


# ------------------------------------------------------------------------------------------------ inputs

def _gen(seed, tag):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + tag * 7919 + 12345) % (1 << 62))
    return g


def _dtype(m):
    return torch.float32 if m.dtype == "f32" else torch.bfloat16


def _weights(m, seed):
    """Random-init parameters in canonical [out, in] layout: matrices N(0, 0.02^2), norm gains near 1, small biases."""
    g, dt = _gen(seed, 1), _dtype(m)

    def mat(*shape):
        return torch.empty(shape, dtype=dt, device=DEV).normal_(0.0, m.weight_std, generator=g)

    def gain():
        return torch.empty(m.d_model, dtype=dt, device=DEV).normal_(1.0, 0.05, generator=g)

    d, f = m.d_model, m.d_ff
    w = {"embed": mat(m.vocab, d), "lm_head": mat(m.vocab, d), "final_norm": gain(),
         "head_w1": mat(m.d_head_hidden, m.d_in), "head_b1": mat(m.d_head_hidden), "head_w2": mat(m.d_head_hidden),
         "head_b2": mat(1)}
    per = {n: [] for n in ("attn_norm", "wq", "wk", "wv", "wo", "ffn_norm", "w_gate", "w_up", "w_down")}
    for _ in range(m.n_layers):
        per["attn_norm"].append(gain())
        per["wq"].append(mat(m.d_q, d))
        per["wk"].append(mat(m.d_kv, d))
        per["wv"].append(mat(m.d_kv, d))
        per["wo"].append(mat(d, m.d_q))
        per["ffn_norm"].append(gain())
        per["w_gate"].append(mat(f, d))
        per["w_up"].append(mat(f, d))
        per["w_down"].append(mat(d, f))
    w.update(per)
    return w


def _lens(case):
    """Cached tokens per stream: a property of the case, the same for every seed (it shapes the outputs)."""
    b, ctx = case["batch"], case["ctx"]
    if case.get("ragged"):
        rng = np.random.default_rng([b, case["k"], ctx])
        return [int(rng.integers(max(1, ctx // 8), ctx + 1)) for _ in range(b)]
    return [ctx] * b


def _inputs(case, seed):
    """Everything of a case that comes from the seed (besides the parameters), on the host unless it is large."""
    rng = np.random.default_rng([int(seed), 77])
    g = _gen(seed, 2)
    if case["kind"] == "ss_rule":
        b, k, v = case["batch"], case["k"], case["vocab"]
        r = b * k
        # a peaked target as a trained decoder gives it, a drafter that approximates it (a quarter of its mass
        # structure perturbed, its tail truncated to zero), and tokens drawn from the drafter
        logits = torch.empty(r, v, device=DEV).normal_(0.0, 3.5, generator=g)
        q = logits.roll(1, 0) + torch.empty(r, v, device=DEV).normal_(0.0, 1.0, generator=g)
        q = torch.softmax(q, 1)
        q[q < 0.25 / v] = 0.0
        q /= q.sum(1, keepdim=True)
        toks = torch.multinomial(q, 1, generator=g).view(-1).to(torch.int32)
        pending = toks.view(b, k)[:, 0].clone()
        if b > 3:
            pending[b // 2] = (pending[b // 2] + 1) % v     # one stream whose block does not start at its pending token
        return {"logits": logits, "q": q, "tokens": toks, "pending": pending,
                "u": torch.rand(r, device=DEV, generator=g) * (1 - 1e-6),
                "v": torch.rand(b, device=DEV, generator=g) * (1 - 1e-6)}
    m = MODELS[case["model"]]
    if case["kind"] == "prefill":
        return {"tokens": rng.integers(0, m.vocab, case["n"]).astype(np.int32)}
    b, k = case["batch"], case["k"]
    r = b * k
    lens = _lens(case)
    drafts = rng.integers(0, m.vocab, r).astype(np.int32)
    pred = rng.integers(0, m.vocab, b).astype(np.int32)
    same = rng.random(b) < 0.7                              # a steady-state block starts at the pending token
    pred[same] = drafts.reshape(b, k)[same, 0]
    inp = {"lens": lens, "drafts": drafts, "pred": pred, "max_ctx": max(lens) + k + 3}
    # cached keys and values at the scale this decoder produces them
    cp = binding.ctx_pad(inp["max_ctx"])
    std = m.weight_std * math.sqrt(m.d_model)
    kv = torch.empty((m.n_layers, b, 2, m.n_kv_heads, cp * m.head_dim), dtype=_dtype(m), device=DEV)
    inp["kv"] = kv.normal_(0.0, std, generator=g)
    if case["kind"] == "ss_round":
        q = torch.softmax(torch.empty(r, m.vocab, device=DEV).normal_(0.0, 1.3, generator=g), 1)
        inp["drafts"] = torch.multinomial(q, 1, generator=g).view(-1).to(torch.int32).cpu().numpy()
        inp["pred"] = inp["drafts"].reshape(b, k)[:, 0].copy()
        inp["q"] = q
        inp["u"] = (rng.random(r) * (1 - 1e-6)).astype(np.float32)
        inp["v"] = (rng.random(b) * (1 - 1e-6)).astype(np.float32)
        return inp
    inp["protos"] = {"fh": [PROTO_FH] * b, "sh": [PROTO_SH] * b,
                     "mixed": [PROTO_FH if i % 2 == 0 else PROTO_SH for i in range(b)]}[case["proto"]]
    # drafts are uniform, so every position but a pending first one is a mismatch: SH streams upload all of those
    rows, row_map = 0, np.full(r, -1, np.int32)
    for i in range(b):
        for j in range(k):
            if inp["protos"][i] == PROTO_FH or j > 0 or drafts[i * k] != pred[i]:
                row_map[i * k + j] = rows
                rows += 1
    inp["hd"] = torch.empty(rows, m.d_draft, dtype=_dtype(m), device=DEV).normal_(0.0, 1.0, generator=g)
    inp["hd_row"] = row_map
    snr = 10.0 * np.log10(10.0 ** 1.5 * -np.log1p(-rng.random(b)) + 1e-3)
    bw = rng.choice([5.0, 10.0, 20.0], b)
    inp["csi"] = np.stack([snr, bw, bw * np.log2(1 + 10 ** (snr / 10)), 5 + 45 * rng.random(b)], 1).astype(np.float32)
    inp["tau"] = np.full(b, 0.45, np.float32)
    return inp


def _spans(lens, k):
    """(first slot, one past the last slot, cached length) of runs of neighbouring slots with equal lengths."""
    at = 0
    for n, run in itertools.groupby(lens):
        c = len(list(run))
        yield at, at + c, n
        at += c


def _appended(kv, m, lens, k):
    """Views of the cache rows a round writes (or 64-bit stand-ins of the same layout)."""
    cp = kv.shape[-1] // m.head_dim
    out = []
    for s0, s1, n in _spans(lens, k):
        out.append(kv[:, s0:s1, 0].view(m.n_layers, s1 - s0, m.n_kv_heads, cp, m.head_dim)[:, :, :, n:n + k])
        vp = kv[:, s0:s1, 1].view(m.n_layers, s1 - s0, m.n_kv_heads, cp // 32, m.head_dim, 32)
        p = n
        while p < n + k:
            e = min(n + k, (p // 32 + 1) * 32)
            out.append(vp[:, :, :, p // 32, :, p % 32:p % 32 + e - p])
            p = e
    return out


def _appended_exact(k_new, v_new, lens, k):
    """The same list from k_new, v_new [layers, batch, kv heads, k, head_dim]."""
    out = []
    for s0, s1, n in _spans(lens, k):
        out.append(k_new[:, s0:s1])
        p = n
        while p < n + k:
            e = min(n + k, (p // 32 + 1) * 32)
            out.append(v_new[:, s0:s1, :, p - n:e - n].transpose(-1, -2))
            p = e
    return out


def _prompt_views(kv, m, n):
    """Views of slot 0's cache rows 0 .. n - 1: keys, whole value blocks, the rest of the last value block."""
    cp = kv.shape[-1] // m.head_dim
    kp = kv[:, 0, 0].view(m.n_layers, m.n_kv_heads, cp, m.head_dim)
    vp = kv[:, 0, 1].view(m.n_layers, m.n_kv_heads, cp // 32, m.head_dim, 32)
    out = [kp[:, :, :n]]
    if n >= 32:
        out.append(vp[:, :, :n // 32])
    if n % 32:
        out.append(vp[:, :, n // 32, :, :n % 32])
    return out


# ------------------------------------------------------------------------------------------------ prepare and run

def prepare(case, seed):
    inp = _inputs(case, seed)
    if case["kind"] == "ss_rule":
        # a context is needed to call the rule; its target plays no part, so the smallest one serves
        m = replace(TINY, n_layers=1, vocab=case["vocab"])
        ctx = binding.Context(m, _weights(m, seed), case["batch"], 32, case["k"])
        b, r = case["batch"], case["batch"] * case["k"]
        out = (torch.zeros(b, dtype=torch.int32, device=DEV), torch.zeros(b, dtype=torch.int32, device=DEV),
               torch.zeros(r, dtype=torch.float32, device=DEV))
        torch.cuda.synchronize()
        return {"case": case, "ctx": ctx, "inp": inp, "out": out}
    m = MODELS[case["model"]]
    if case["kind"] == "prefill":
        max_ctx = case["n"] + case["k"] + 3
        kv = binding.new_kv_cache(m, case["batch"], max_ctx, DEV)
        ctx = binding.Context(m, _weights(m, seed), case["batch"], max_ctx, case["k"], kv_cache=kv)
        return {"case": case, "ctx": ctx, "inp": inp, "kv": kv, "views": _prompt_views(kv, m, case["n"])}
    b, k = case["batch"], case["k"]
    ctx = binding.Context(m, _weights(m, seed), b, inp["max_ctx"], k, kv_cache=inp["kv"])
    for s in range(b):
        ctx.wisv_set_state(s, inp["lens"][s], int(inp["pred"][s]))
    st = {"case": case, "ctx": ctx, "inp": inp, "sid": np.arange(b, dtype=np.int32),
          "views": _appended(inp["kv"], m, inp["lens"], k)}
    nc = binding.WISV_FLAG_NO_COMMIT                        # so that the pass can be repeated on the same state
    if case["kind"] == "ss_round":
        st["round"] = ctx.ss_device_round(st["sid"], inp["drafts"], inp["q"], inp["u"], inp["v"], k, nc)
        return st
    call = case["call"]
    if call in ("device", "logits"):
        st["round"] = ctx.device_round(st["sid"], inp["drafts"], inp["protos"], inp["hd"], inp["hd_row"], inp["csi"],
                                       inp["tau"], k, nc | (binding.WISV_FLAG_KEEP_LOGITS if call == "logits" else 0))
    else:
        inp["hd"] = inp["hd"].cpu()                         # an uploaded row arrives in host memory
    torch.cuda.synchronize()
    return st


def run(state):
    case, ctx, inp = state["case"], state["ctx"], state["inp"]
    kind, k = case["kind"], case["k"]
    if kind == "ss_rule":
        return list(ctx.wisv_ss_decide(inp["logits"], inp["pending"], inp["tokens"], inp["q"], inp["u"], inp["v"], k,
                                       out=state["out"]))
    if kind == "prefill":
        ctx.wisv_set_state(0, 0, 0)                         # the slot is handed to a new request
        ctx.wisv_prefill(0, inp["tokens"])
        return {"state": list(ctx.wisv_get_state(0)), "kv": state["views"]}
    if kind == "ss_round":
        state["round"].run()
        o = state["round"].out
        return {"round": [o[n] for n in ("accepted_len", "correction_token", "alpha")], "kv": state["views"]}
    names = ("accepted_len", "correction_token", "p_accept", "target_argmax", "mismatch_mask", "status")
    nc = binding.WISV_FLAG_NO_COMMIT
    call, rows = case["call"], case["batch"] * k
    if call in ("device", "logits"):
        state["round"].run()
        o = state["round"].out
        res = {"round": [o[n] for n in names], "kv": state["views"]}
        if call == "logits":
            res["logits"] = ctx.wisv_debug_copy(binding.WISV_DBG_LOGITS, rows)
        return res
    args = (inp["csi"], inp["tau"], k)
    if call == "two":
        first = ctx.wisv_verify_round(state["sid"], inp["drafts"], inp["protos"], None, np.full(rows, -1, np.int32), *args,
                                      binding.WISV_FLAG_VERIFY_ONLY)
        o = ctx.wisv_verify_round(state["sid"], inp["drafts"], inp["protos"], inp["hd"], inp["hd_row"], *args,
                                  binding.WISV_FLAG_DECIDE_ONLY | nc)
        return {"request": [first[n].reshape(-1) for n in ("target_argmax", "mismatch_mask")],
                "round": [o[n].reshape(-1) for n in names], "kv": state["views"]}
    keep = binding.WISV_FLAG_KEEP_LOGITS if call == "host_logits" else 0
    o = ctx.wisv_verify_round(state["sid"], inp["drafts"], inp["protos"], inp["hd"], inp["hd_row"], *args, nc | keep)
    res = {"round": [o[n].reshape(-1) for n in names], "kv": state["views"]}
    if keep:
        res["logits"] = ctx.wisv_debug_copy(binding.WISV_DBG_LOGITS, rows)
    return res


# ------------------------------------------------------------------------------------------------ work and tolerance

def work(case):
    if case["kind"] == "ss_rule":
        # every logits row once, one drafter row per stream (the residual), a multiply and an exponential per logit
        r, v = case["batch"] * case["k"], case["vocab"]
        return {"bytes": (r + case["batch"]) * v * 4, "flops": 4 * r * v}
    m = MODELS[case["model"]]
    e = 4 if m.dtype == "f32" else 2
    layers = m.n_layers * m.layer_params()
    head = m.vocab * m.d_model
    if case["kind"] == "prefill":
        n = case["n"]
        return {"bytes": e * (layers + head) + n * m.kv_bytes_per_token(),
                "flops": 2 * n * layers + 2 * head + m.n_layers * 4 * m.d_q * (n * (n + 1) // 2)}
    r = case["batch"] * case["k"]
    toks = sum(_lens(case))
    mean = toks / case["batch"]
    w = {"bytes": e * (layers + head) + (toks + r) * m.kv_bytes_per_token(),
         "flops": 2 * r * (layers + head) + int(m.n_layers * 4 * m.d_q * r * mean)}
    if case["kind"] == "ss_round":
        w["bytes"] += case["batch"] * m.vocab * 4
    else:
        w["bytes"] += m.head_bytes() + r * m.d_draft * e
        w["flops"] += 2 * r * m.d_head_hidden * m.d_in
        if "logits" in case["call"]:
            w["bytes"] += r * m.vocab * 4
    return w


def tolerance(case):
    """About four times what the path shows against 64 bits, by what bounds its precision: 32-bit sums for the fp32
    target and the sampling rule; for the bf16 target one step of the 16-bit cache wherever a key or value sits at a
    rounding boundary (4e-4 to 7e-4 with two-term activations), and the half-precision activations of rounds of more
    than 16 rows (1.2e-3).  Whole numbers follow from comparisons (an argmax over 32000 tokens, a probability against
    a threshold): one stream's may turn on a near tie."""
    if case["kind"] == "ss_rule":
        return {"rel": 1e-6, "max": 1e-5, "differ": min(0.5, max(0.02, 1.01 / case["batch"]))}
    if case["model"] == "tiny":
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}
    one_term = case["batch"] * case["k"] > 16
    rel = 5e-3 if one_term else 3e-3 if case["kind"] == "prefill" else 2e-3
    return {"rel": rel, "max": 10 * rel, "differ": min(0.5, max(0.05, 1.01 / case["batch"]))}


# ------------------------------------------------------------------------------------------------ 64 bits

def _rms(x, g, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * g.double()


def _rope(x, pos, theta):
    """x [rows, heads, head_dim] at positions pos [rows], rotate-half pairing."""
    half = x.shape[-1] // 2
    inv = theta ** (-torch.arange(half, device=DEV, dtype=torch.float64) * 2 / x.shape[-1])
    a = pos.double()[:, None, None] * inv
    c, s = torch.cos(a), torch.sin(a)
    return torch.cat([x[..., :half] * c - x[..., half:] * s, x[..., half:] * c + x[..., :half] * s], -1)


def _forward(m, w, tokens, lens, k, kv):
    """The decoder in 64 bits over len(lens) streams of k tokens each after lens[b] cached ones (kv: the cache tensor, or
    None when nothing is cached).  The cache stores the model's type: k and v are rounded to it where it is 16 bits
    wide.  Returns (final hidden states, new keys, new values [layers, batch, kv heads, k, head_dim])."""
    b, hd, nh, ng = len(lens), m.head_dim, m.n_heads, m.n_kv_heads
    store = (lambda t: t.to(torch.bfloat16).double()) if m.dtype != "f32" else (lambda t: t)
    pos = torch.cat([torch.arange(n, n + k, device=DEV) for n in lens])
    x = w["embed"][torch.as_tensor(tokens, device=DEV).long()].double()
    new_k, new_v = [], []
    tri = torch.ones(k, k, device=DEV, dtype=torch.bool).triu(1)
    for l in range(m.n_layers):
        a = _rms(x, w["attn_norm"][l], m.rms_eps)
        q = _rope((a @ w["wq"][l].double().t()).view(-1, nh, hd), pos, m.rope_theta)
        kn = store(_rope((a @ w["wk"][l].double().t()).view(-1, ng, hd), pos, m.rope_theta))
        vn = store((a @ w["wv"][l].double().t()).view(-1, ng, hd))
        new_k.append(kn.view(b, k, ng, hd).transpose(1, 2))
        new_v.append(vn.view(b, k, ng, hd).transpose(1, 2))
        o = torch.empty_like(q)
        for i, n in enumerate(lens):
            rows = slice(i * k, (i + 1) * k)
            ks, vs = new_k[-1][i], new_v[-1][i]
            if n:
                cp = kv.shape[-1] // hd
                ks = torch.cat([kv[l, i, 0].view(ng, cp, hd)[:, :n].double(), ks], 1)
                vc = kv[l, i, 1].view(ng, cp // 32, hd, 32)[:, :(n + 31) // 32]
                vs = torch.cat([vc.transpose(2, 3).reshape(ng, -1, hd)[:, :n].double(), vs], 1)
            for h in range(ng):
                rep = nh // ng
                qh = q[rows, h * rep:(h + 1) * rep]                       # [k, rep, hd]
                s = torch.matmul(qh.reshape(-1, hd), ks[h].t().contiguous()).view(k, rep, n + k) / math.sqrt(hd)
                s[:, :, n:].masked_fill_(tri[:, None, :], -math.inf)
                o[rows, h * rep:(h + 1) * rep] = torch.matmul(torch.softmax(s, -1).view(-1, n + k), vs[h]).view(k, rep, hd)
        x = x + o.reshape(-1, m.d_q) @ w["wo"][l].double().t()
        a = _rms(x, w["ffn_norm"][l], m.rms_eps)
        gt = a @ w["w_gate"][l].double().t()
        x = x + (gt / (1 + torch.exp(-gt)) * (a @ w["w_up"][l].double().t())) @ w["w_down"][l].double().t()
    return _rms(x, w["final_norm"], m.rms_eps), torch.stack(new_k), torch.stack(new_v)


def _ss_exact(logits, q, tokens, pending, u, v, b, k):
    """The rule of speculative sampling in 64 bits: accepted lengths, emitted tokens, acceptance probabilities."""
    p = torch.softmax(logits.double(), 1)
    q = q.double()
    tok = torch.as_tensor(tokens, device=DEV).long()
    al = torch.empty(b, k, dtype=torch.float64, device=DEV)
    al[:, 0] = (tok.view(b, k)[:, 0] == torch.as_tensor(pending, device=DEV).long()).double()
    if k > 1:
        idx = torch.arange(b * k, device=DEV).view(b, k)[:, 1:].reshape(-1)
        pt, qt = p[idx - 1, tok[idx]], q[idx, tok[idx]]
        al[:, 1:] = torch.where(qt <= pt, torch.ones_like(pt), pt / qt.clamp_min(1e-300)).view(b, k - 1)
    rej = ~(torch.as_tensor(u, device=DEV).double().view(b, k) < al)
    pos = torch.arange(k, device=DEV).expand(b, k)
    a = torch.where(rej, pos, torch.full_like(pos, k)).min(1).values
    emit = torch.empty(b, dtype=torch.long, device=DEV)
    vv = torch.as_tensor(v, device=DEV).double()
    for i in range(b):
        n = int(a[i])
        if n == 0:
            emit[i] = int(pending[i])
            continue
        row = i * k + n - 1
        wt = (p[row] - q[row + 1]).clamp_min(0) if n < k else p[row]
        cum = wt.cumsum(0)
        hit = torch.nonzero((cum > vv[i] * cum[-1]) & (wt > 0))
        emit[i] = hit[0, 0] if hit.numel() else torch.nonzero(wt > 0)[-1, 0]
    return [a, emit, al.reshape(-1)]


def exact(case, seed):
    inp = _inputs(case, seed)
    if case["kind"] == "ss_rule":
        r = _ss_exact(inp["logits"], inp["q"], inp["tokens"], inp["pending"], inp["u"], inp["v"], case["batch"], case["k"])
        return [r[0], r[1], r[2].view(case["batch"], case["k"])]
    m = MODELS[case["model"]]
    w = _weights(m, seed)
    k = case["k"]
    if case["kind"] == "prefill":
        n = case["n"]
        h, kn, vn = _forward(m, w, inp["tokens"], [0], n, None)
        nxt = int((w["lm_head"].double() @ h[-1]).argmax())
        kn, vn = kn[:, 0], vn[:, 0]
        kv = [kn]
        if n >= 32:
            kv.append(vn[:, :, :n // 32 * 32].reshape(m.n_layers, m.n_kv_heads, n // 32, 32, m.head_dim).transpose(3, 4))
        if n % 32:
            kv.append(vn[:, :, n // 32 * 32:].transpose(2, 3))
        return {"state": [n, nxt], "kv": kv}
    b, lens = case["batch"], inp["lens"]
    h, kn, vn = _forward(m, w, inp["drafts"], lens, k, inp["kv"])
    kv = _appended_exact(kn, vn, lens, k)
    logits = h @ w["lm_head"].double().t()
    if case["kind"] == "ss_round":
        return {"round": _ss_exact(logits, inp["q"], inp["drafts"], inp["pred"], inp["u"], inp["v"], b, k), "kv": kv}
    amax = logits.argmax(1).view(b, k)
    pred = torch.as_tensor(inp["pred"], device=DEV).long()
    tgt = torch.cat([pred[:, None], amax], 1)
    mis = torch.as_tensor(inp["drafts"], device=DEV).long().view(b, k) != tgt[:, :k]
    row = torch.as_tensor(inp["hd_row"], device=DEV).long()
    hd = inp["hd"].to(DEV).double()[row.clamp_min(0)]
    csi = torch.as_tensor(inp["csi"], device=DEV).double().repeat_interleave(k, 0)
    z = torch.cat([hd, h, csi], 1)
    a1 = z @ w["head_w1"].double().t() + w["head_b1"].double()
    s = (a1 / (1 + torch.exp(-a1))) @ w["head_w2"].double() + w["head_b2"].double()
    fh = torch.tensor([p == PROTO_FH for p in inp["protos"]], device=DEV)[:, None]
    scored = (fh | mis) & (row.view(b, k) >= 0)
    p = torch.where(scored, 1 / (1 + torch.exp(s.view(b, k))), torch.ones(b, k, dtype=torch.float64, device=DEV))
    tau = torch.as_tensor(inp["tau"], device=DEV).double()[:, None]
    rej = mis & (~scored | ~(p >= tau))
    pos = torch.arange(k, device=DEV).expand(b, k)
    a = torch.where(rej, pos, torch.full_like(pos, k)).min(1).values
    y = tgt.gather(1, a[:, None])[:, 0]
    mask = (mis.long() << pos).sum(1)
    status = (mis & ~scored).any(1).long()
    res = {"round": [a, y, p.reshape(-1), tgt.reshape(-1), mask, status], "kv": kv}
    if case["call"] == "two":
        res["request"] = [tgt.reshape(-1), mask]
    if "logits" in case["call"]:
        res["logits"] = logits
    return res
