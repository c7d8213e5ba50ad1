"""The work that a program has this library do, as cases for timing and comparison.

A case is a dict of plain values; `kind` names the public entry point it goes through:

  proj         amd.gemm: one decode-time projection of 1..32 new tokens (QKV, O, gate/up, down or LM head of a layer)
  prompt_proj  amd.dense_gemm: one prompt-time projection, plain (epilogue 0) or with SiLU * mul (epilogue 2)
  sample       amd.sample_row: a draft model's distribution and draw from one row of logits
  accept       amd.accept_rows_static: acceptance of a window of drafts, resampling and bonus token included
  forward      SpecContext.verify: a forward over M new tokens against a filled K/V cache, then the rollback of them
  prompt       SpecContext.prefill + verify: a prompt pass and the first row of logits after it
  pearl        SpecContext.generate: the whole parallel speculative decoding loop, two models on two streams

Widths are those of synth.config's pairs, depths are cut where a whole model would not fit the GPU three times.  Matrices
are N(0, s^2) with s = min(0.02, 0.9 / sqrt(fan-in)): at 0.02 the wide random-init models amplify a rounding error from
layer to layer, which trained ones do not.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2408_11850_amd as amd
from paper_2408_11850_amd import harness

synth = harness.synth
PAIRS = ("tiny", "small", "7b_1b", "33b_1b", "70b_7b")


def listed():
    return [
        # the output projection of a 1B-shape draft model: the smallest matrix of a decode step, one token, all latency
        {"name": "proj_1b_o_m1", "kind": "proj", "m": 1, "n": 2048, "k": 2048},
        # the down projection of the 70B-shape target over a verify window of 7: the ordinary large decode matrix
        {"name": "proj_70b_down_m7", "kind": "proj", "m": 7, "n": 8192, "k": 28672},
        # gate/up of the 33B-shape target with the largest adaptive window, 16 drafts and the frontier: two row tiles
        {"name": "proj_33b_gateup_m17", "kind": "proj", "m": 17, "n": 38400, "k": 7168},
        # QKV of the small pair for its 512-token prompt (the last token is not part of the prompt pass)
        {"name": "prompt_small_qkv", "kind": "prompt_proj", "m": 511, "n": 6144, "k": 2048, "epilogue": 0},
        # gate/up of the 70B-shape target for its 4096-token prompt: the largest single call there is
        {"name": "prompt_70b_gateup", "kind": "prompt_proj", "m": 4095, "n": 57344, "k": 8192, "epilogue": 2},
        # a draft step's draw at the pairs' vocabulary
        {"name": "sample_32000", "kind": "sample", "v": 32000, "temperature": 1.0},
        # acceptance of an SD window of 7 at the vocabulary of the larger tokenizers (beyond 32768 ids)
        {"name": "accept_128256", "kind": "accept", "v": 128256, "rows": 8, "tests": 7, "temperature": 1.0},
        # a draft step's forward on the 7B shape behind the benchmark's prompt: one token, four layers, LM head
        {"name": "decode_7b_m1", "kind": "forward", "pair": "70b_7b", "model": "draft", "depth": 4, "context": 4096, "m": 1},
        # the verify forward of the 70B shape over the benchmark's window, four layers, LM head
        {"name": "verify_70b_m7", "kind": "forward", "pair": "70b_7b", "model": "target", "depth": 4, "context": 4096, "m": 7},
        # the small pair's target as a whole (24 layers), the verify forward of a window of 4 and a bonus row
        {"name": "verify_small_m5", "kind": "forward", "pair": "small", "model": "target", "depth": 24, "context": 512, "m": 5},
        # a 1024-token prompt through layers of the 7B shape up to the first row of logits
        {"name": "prompt_7b_1024", "kind": "prompt", "pair": "7b_1b", "model": "target", "depth": 4, "tokens": 1024},
        # the whole loop on the small pair: 64 greedy tokens with windows of 4, a draft that is right about 6 times in 7
        {"name": "pearl_small_g4", "kind": "pearl", "pair": "small", "depth": 24, "draft_depth": 4, "context": 512, "gamma": 4,
         "tokens": 64},
    ]


def _log_int(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi + 0.999 * step)))
    return max(lo, min(hi, int(v) // step * step))


def _shape(case):
    cfg = synth.config(case["pair"])
    s = cfg.draft if case.get("model") == "draft" else cfg.target
    return synth._truncate(s, min(case["depth"], s.n_layers))


def draw(rng):
    most = {c["name"]: work(c) for c in listed()}
    kind = rng.choice(["proj", "proj", "prompt_proj", "prompt_proj", "sample", "accept", "forward", "forward", "forward",
                       "prompt", "prompt", "pearl"])
    while True:
        if kind == "proj":
            c = {"kind": kind, "m": _log_int(rng, 1, 32), "n": _log_int(rng, 256, 57344, 16), "k": _log_int(rng, 256, 28672, 8)}
            if c["n"] * c["k"] > 57344 * 8192:
                continue
        elif kind == "prompt_proj":
            c = {"kind": kind, "m": _log_int(rng, 65, 4096), "n": _log_int(rng, 512, 57344, 32),
                 "k": _log_int(rng, 512, 28672, 32), "epilogue": rng.choice([0, 2])}
            if work(c)["flops"] > most["prompt_70b_gateup"]["flops"] or c["m"] * c["n"] > 1 << 28:
                continue
        elif kind == "sample":
            c = {"kind": kind, "v": _log_int(rng, 1024, 131072), "temperature": rng.choice([1.0, 0.7, 0.0])}
        elif kind == "accept":
            t = rng.randint(1, 16)
            c = {"kind": kind, "v": _log_int(rng, 1024, 131072), "rows": t + rng.randint(0, 1), "tests": t,
                 "temperature": rng.choice([1.0, 0.7, 0.0])}
        elif kind == "forward":
            c = {"kind": kind, "pair": rng.choice(PAIRS), "model": rng.choice(["target", "draft"]), "depth": rng.randint(1, 8),
                 "context": _log_int(rng, 17, 4096), "m": _log_int(rng, 1, 32)}
            if work(c)["bytes"] > most["verify_70b_m7"]["bytes"]:
                continue
        elif kind == "prompt":
            c = {"kind": kind, "pair": rng.choice(PAIRS), "model": rng.choice(["target", "draft"]), "depth": rng.randint(1, 8),
                 "tokens": _log_int(rng, 66, 4096)}
            if work(c)["flops"] > most["prompt_70b_gateup"]["flops"]:
                continue
        else:
            c = {"kind": kind, "pair": "small", "depth": rng.randint(8, 24), "draft_depth": rng.randint(1, 4),
                 "context": _log_int(rng, 33, 1024), "gamma": rng.randint(1, 8), "tokens": rng.randint(16, 64)}
        return c


# ---- inputs ---------------------------------------------------------------------------------------------------------
_SLOTS = {"wq": 0, "wk": 1, "wv": 2, "wo": 3, "w_gate": 4, "w_up": 5, "w_down": 6, "attn_norm": 7, "ffn_norm": 8,
          "tok_embed": 9, "lm_head": 10, "final_norm": 11, "x": 12, "w": 13, "logits": 14, "q": 15}


def _normal(shape, std, seed, name, layer=0, dtype=torch.bfloat16, mean=0.0):
    gen = torch.Generator(device="cuda")
    gen.manual_seed((int(seed) * 4096 + layer) * 16 + _SLOTS[name])
    return torch.empty(shape, dtype=torch.float32, device="cuda").normal_(mean, std, generator=gen).to(dtype)


def _std(fan_in):
    return min(0.02, 0.9 / math.sqrt(fan_in))


def _ints(n, top, seed, salt):
    gen = torch.Generator()
    gen.manual_seed(int(seed) * 16 + salt)
    return torch.randint(0, top, (n,), generator=gen).tolist()


def _tensor(s, seed, layer, name):
    """One bf16 tensor of a model, row-major, as the packing takes it."""
    if name in ("final_norm", "attn_norm", "ffn_norm"):
        return _normal((s.d_model,), synth.GAIN_STD, seed, name, layer or 0, mean=1.0)
    shape = (s.vocab, s.d_model) if layer is None else synth.layer_matrix_shapes(s)[name]
    return _normal(shape, _std(shape[1]), seed, name, layer or 0)


def _succession(v, seed):
    """(next id under the target, next id under the draft model) for every id: two permutations that agree on 6 of 7 ids."""
    gen = torch.Generator()
    gen.manual_seed(int(seed) * 16 + 5)
    nxt = torch.randperm(v, generator=gen)
    other = torch.randperm(v, generator=gen)[: v // 7]
    drafted = nxt.clone()
    drafted[other] = nxt[other.roll(1)]
    return nxt, drafted


def _pearl_tensor(s, seed, layer, name, drafted=False):
    """As _tensor, with an embedding of unit variance and an LM head that answers an id's own embedding with its successor:
    greedy decisions are then as clear as a trained model's, and the rate of accepted drafts is as high."""
    if name == "tok_embed":
        return _normal((s.vocab, s.d_model), 1.0, seed, name)
    if name == "lm_head":
        e = _normal((s.vocab, s.d_model), 1.0, seed, "tok_embed")
        head = torch.empty_like(e)
        head[_succession(s.vocab, seed)[1 if drafted else 0].cuda()] = e * 2.0 ** -6
        return head
    return _tensor(s, seed, layer, name)


def _logit_rows(case, seed):
    """Target logits and draft distributions of an acceptance: peaked rows, the draft's close to the target's."""
    v, rows, tests = case["v"], case["rows"], case["tests"]
    p = _normal((rows, v), 3.0, seed, "logits", dtype=torch.float32)
    ql = p[:tests] + _normal((tests, v), 0.3, seed, "q", dtype=torch.float32)
    if case["temperature"] == 0.0:
        q = torch.zeros_like(ql)
        q[torch.arange(tests, device="cuda"), ql.argmax(-1)] = 1.0
        x = ql.argmax(-1)
    else:
        q = torch.softmax(ql.double() / case["temperature"], -1).float()
        u = torch.tensor(_uniforms(tests, seed, 6), device="cuda", dtype=torch.float64)
        x = torch.searchsorted(q.double().cumsum(-1), u[:, None]).clamp(max=v - 1)[:, 0]
    return p.contiguous(), q.contiguous(), x.to(torch.int32)


def _uniforms(n, seed, salt):
    return [(2 * i + 1) / 16777216.0 for i in _ints(n, 1 << 23, seed, salt)]


# Both sides of a context's life: max_seq holds the prompt, the new tokens and the ring of drafts.
def _context(s, seed, room):
    target = amd.pack_model(s, lambda layer, name: _tensor(s, seed, layer, name))
    draft = target.prefix(1, synth._truncate(s, 1))
    return amd.SpecContext(target, draft, gamma_max=amd.SPEC_MAX_TOKENS - 1, max_seq=room + 4 * amd.SPEC_MAX_TOKENS)


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("proj", "prompt_proj"):
        w = _normal((case["n"], case["k"]), _std(case["k"]), seed, "w")
        packed = amd.binding.pack_matrices([w])
        return {"case": case, "x": _normal((case["m"], case["k"]), 1.0, seed, "x"), "w": packed}
    if kind == "sample":
        row = _normal((case["v"],), 3.0, seed, "logits", dtype=torch.float32)
        return {"case": case, "row": row, "u": _uniforms(1, seed, 3)[0]}
    if kind == "accept":
        p, q, x = _logit_rows(case, seed)
        u = _uniforms(case["tests"] + 1, seed, 4)
        return {"case": case, "p": p, "q": q, "x": x, "r": np.asarray(u[:-1], np.float32), "u": u[-1],
                "result": torch.zeros(2, dtype=torch.int32, device="cuda")}
    if kind == "pearl":
        cfg, target, draft = _pearl_models(case, seed)
        prompt = _ints(case["context"], cfg.target.vocab, seed, 1)
        ctx = harness.make_context(cfg, target, draft, case["gamma"])
        ctx.prefill(prompt)
        return {"case": case, "ctx": ctx, "prompt": prompt, "uniforms": synth.make_uniforms(case["tokens"] + 1, case["gamma"], seed)}
    s = _shape(case)
    if kind == "prompt":
        return {"case": case, "ctx": _context(s, seed, case["tokens"]), "prompt": _ints(case["tokens"], s.vocab, seed, 1)}
    prompt = _ints(case["context"] + 1, s.vocab, seed, 1)
    ctx = _context(s, seed, case["context"] + 1)
    ctx.prefill(prompt, which_mask=1)
    return {"case": case, "ctx": ctx, "new": prompt[-1:] + _ints(case["m"] - 1, s.vocab, seed, 2)}


def _pearl_models(case, seed):
    base = synth.config(case["pair"], depth=case["depth"], draft_depth=case["draft_depth"])
    s = base.target
    target = amd.pack_model(s, lambda layer, name: _pearl_tensor(s, seed, layer, name))
    draft = target.prefix(case["draft_depth"], base.draft)
    draft.lm_head = amd.binding.pack_matrices([_pearl_tensor(s, seed, None, "lm_head", drafted=True)])
    torch.cuda.synchronize()
    base.n_prompt, base.n_generate, base.temperature, base.gamma = case["context"], case["tokens"], 0.0, case["gamma"]
    return base, target, draft


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "proj":
        return amd.gemm(state["x"], state["w"], case["n"])
    if kind == "prompt_proj":
        return amd.dense_gemm(state["x"], state["w"], case["n"], case["epilogue"])
    if kind == "sample":
        return amd.sample_row(state["row"], case["temperature"], 1.0, state["u"])
    if kind == "accept":
        amd.accept_rows_static(state["p"], state["q"], state["x"], state["r"], case["temperature"], 1.0, state["u"],
                               state["result"])
        return state["result"]
    ctx = state["ctx"]
    if kind == "forward":
        logits = ctx.verify(state["new"], want_logits=True)
        ctx.rollback_kv(amd.SPEC_TARGET, case["context"])
        return logits
    if kind == "prompt":
        ctx.prefill(state["prompt"], which_mask=1)
        return ctx.verify(state["prompt"][-1:], want_logits=True)
    # another answer to the same prompt: back to it, decode, and the logits that follow the last token
    ctx.rewind(len(state["prompt"]))
    tokens, _ = ctx.generate(amd.ALGO_PEARL, case["gamma"], case["tokens"], state["uniforms"])
    ctx.rewind(len(state["prompt"]) + case["tokens"])
    return np.asarray(tokens, np.int64), ctx.verify(tokens[-1:], want_logits=True)


# ---- what a pass cannot do without ----------------------------------------------------------------------------------
def _forward_work(s, rows, context, logit_rows):
    """A forward over `rows` tokens behind `context`: every weight once, the cache once, the new K/V rows and the logits."""
    layer = s.params_per_layer() * s.n_layers
    head = s.vocab * s.d_model if logit_rows else 0
    seen = rows * context + rows * (rows + 1) // 2
    return {"bytes": 2 * (layer + head) + (context + rows) * s.kv_bytes_per_token() + 4 * logit_rows * s.vocab,
            "flops": 2 * rows * layer + 2 * logit_rows * head + 4 * seen * s.n_layers * s.n_heads * s.head_dim}


def _sum(parts):
    return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}


def work(case):
    kind = case["kind"]
    if kind in ("proj", "prompt_proj"):
        m, n, k = case["m"], case["n"], case["k"]
        out = 2 * m * (n // 2) if case.get("epilogue") == 2 else 4 * m * n
        return {"bytes": 2 * n * k + 2 * m * k + out, "flops": 2 * m * n * k}
    if kind == "sample":
        return {"bytes": 8 * case["v"], "flops": 6 * case["v"]}
    if kind == "accept":   # every target row for its normaliser, one draft row for the residual
        return {"bytes": 4 * case["v"] * (case["rows"] + 1), "flops": 6 * case["v"] * case["rows"]}
    if kind == "forward":
        return _forward_work(_shape(case), case["m"], case["context"], case["m"])
    if kind == "prompt":
        s = _shape(case)
        return _sum([_forward_work(s, case["tokens"] - 1, 0, 0), _forward_work(s, 1, case["tokens"] - 1, 1)])
    # at best every draft is accepted: a target forward per window, a draft forward per token
    cfg = synth.config(case["pair"], depth=case["depth"], draft_depth=case["draft_depth"])
    t, d = cfg.target, cfg.draft
    windows = -(-case["tokens"] // case["gamma"])
    return _sum([_forward_work(t, case["gamma"], case["context"], case["gamma"])] * windows
                + [_forward_work(d, 1, case["context"], 1)] * case["tokens"] + [_forward_work(t, 1, case["context"], 1)])


def tolerance(case):
    kind = case["kind"]
    if kind == "proj" or (kind == "prompt_proj" and case["epilogue"] == 0):
        return {"rel": 1e-5, "max": 1e-4}
    if kind == "prompt_proj":
        return {"rel": 4e-3, "max": 2e-2}   # one bf16 rounding of the product
    if kind == "sample":
        return {"rel": 1e-5, "max": 1e-4}
    if kind == "accept":
        return "exact"
    # two correct prompt passes (one dense block, or blocks of 32 tokens) leave logits 1.0e-2 apart, at most 0.05
    return {"rel": 3e-2, "max": 0.2}


# ---- the same in 64 bits, in plain torch -----------------------------------------------------------------------------
def _rope(x, theta):
    t, _, d = x.shape
    half = d // 2
    ang = torch.arange(t, device="cuda", dtype=torch.float64)[:, None] * \
        theta ** (-2.0 * torch.arange(half, device="cuda", dtype=torch.float64) / d)
    c, s = ang.cos()[:, None, :], ang.sin()[:, None, :]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, a * s + b * c], -1)


def _norm(h, gain, eps):
    return h / (h.square().mean(-1, keepdim=True) + eps).sqrt() * gain


def _exact_logits(s, get, tokens, rows):
    """Logits of the last `rows` of `tokens`, one forward over all of them."""
    w = lambda layer, name: get(layer, name).double()  # noqa: E731
    h = w(None, "tok_embed")[torch.tensor(tokens, device="cuda")]
    t, hq, hkv, d = len(tokens), s.n_heads, s.n_kv_heads, s.head_dim
    hidden = torch.ones((t, t), dtype=torch.bool, device="cuda").triu_(1)
    for layer in range(s.n_layers):
        a = _norm(h, w(layer, "attn_norm"), s.rms_eps)
        q = _rope((a @ w(layer, "wq").T).view(t, hq, d), s.rope_theta)
        k = _rope((a @ w(layer, "wk").T).view(t, hkv, d), s.rope_theta)
        v = (a @ w(layer, "wv").T).view(t, hkv, d)
        o = torch.empty_like(q)
        for i in range(hq):
            j = i // (hq // hkv)
            score = (q[:, i] @ k[:, j].T) / math.sqrt(d)
            o[:, i] = score.masked_fill_(hidden, -math.inf).softmax(-1) @ v[:, j]
        h = h + o.view(t, hq * d) @ w(layer, "wo").T
        a = _norm(h, w(layer, "ffn_norm"), s.rms_eps)
        h = h + (torch.nn.functional.silu(a @ w(layer, "w_gate").T) * (a @ w(layer, "w_up").T)) @ w(layer, "w_down").T
    return _norm(h[-rows:], w(None, "final_norm"), s.rms_eps) @ w(None, "lm_head").T


def exact(case, seed):
    kind = case["kind"]
    if kind in ("proj", "prompt_proj"):
        w = _normal((case["n"], case["k"]), _std(case["k"]), seed, "w")
        y = _normal((case["m"], case["k"]), 1.0, seed, "x").double() @ w.double().T
        if case.get("epilogue") != 2:
            return y
        y = y.view(case["m"], -1, 2, 16)   # panels of 16 columns: gate, up, gate, up ..
        return (torch.nn.functional.silu(y[:, :, 0]) * y[:, :, 1]).reshape(case["m"], -1)
    if kind == "sample":
        if case["temperature"] == 0.0:
            return None
        row = _normal((case["v"],), 3.0, seed, "logits", dtype=torch.float32)
        return torch.softmax(row.double() / case["temperature"], -1), None
    if kind == "accept":
        return None
    if kind == "pearl":
        cfg = synth.config(case["pair"], depth=case["depth"], draft_depth=case["draft_depth"])
        s = cfg.target
        tokens = _ints(case["context"], s.vocab, seed, 1)
        nxt = _succession(s.vocab, seed)[0].tolist()
        for _ in range(case["tokens"]):
            tokens.append(nxt[tokens[-1]])
        made = np.asarray(tokens[case["context"]:], np.int64)
        return made, _exact_logits(s, lambda layer, name: _pearl_tensor(s, seed, layer, name), tokens, 1)
    s = _shape(case)
    if kind == "prompt":
        tokens, rows = _ints(case["tokens"], s.vocab, seed, 1), 1
    else:
        tokens = _ints(case["context"] + 1, s.vocab, seed, 1) + _ints(case["m"] - 1, s.vocab, seed, 2)
        rows = case["m"]
    return _exact_logits(s, lambda layer, name: _tensor(s, seed, layer, name), tokens, rows)
