"""The calls that a program on this library makes, at the sizes it makes them with.

Two kinds of case.  ``attention`` is one scheduling iteration of one layer: ``Handle.kv_append`` of the batch's new
keys and values, then ``Handle.hybrid_attention`` (or its allocation-free form) over prefill chunks and decodes.
``linear`` is the four linear layers of one transformer layer over the batch's tokens, through ``binding.linear``.
Shapes are those of the models in ``linear_layers.MODELS`` (whole attention heads, or one GPU's share of them under the
model's tensor-parallel degree) and of ``workloads``; ``prepare`` makes tensors on the GPU from the seed alone.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2403_02310_amd import binding, linear_layers, workloads

PAGE = workloads.PAGE_SIZE

# query heads, key/value heads, head_dim
HEADS = {
    "tiny": (4, 1, 64),
    "mistral-7b": (32, 8, 128),
    "yi-34b": (56, 8, 128),
    "llama2-70b": (64, 8, 128),
    "llama2-70b/tp4": (16, 2, 128),
    "falcon-180b/tp4": (58, 2, 64),
}


def _attention(name, heads, chunks="", decodes=0, low=0, high=0, spread="uniform", lengths=0, window=0, entry="workspace"):
    """``chunks``: new tokens @ cached prefix, comma separated.  ``decodes`` sequences of ``low`` to ``high`` keys."""
    return {"name": name, "kind": "attention", "heads": heads, "chunks": chunks, "decodes": decodes, "low": low,
            "high": high, "spread": spread, "lengths": lengths, "window": window, "entry": entry}


def _linear(name, model, tokens):
    return {"name": name, "kind": "linear", "model": model, "tokens": tokens}


def listed():
    return [
        # The smallest call: a short prompt's chunk next to three decodes, one key/value head of 64 channels, through the
        # entry point of programs that hand no workspace over; launches and host time.
        _attention("tiny_hybrid", "tiny", "64@128", 3, 100, 300, lengths=1, entry="noalloc"),
        # A lightly loaded server: eight requests generate, nothing is prefilled.
        _attention("mistral_8_decodes", "mistral-7b", "", 8, 256, 4096, lengths=2),
        # A decode-only iteration of a busy server, skewed context lengths.
        _attention("mistral_256_decodes", "mistral-7b", "", 256, 64, 8192, "lognormal", lengths=3),
        # Stall-free batching's usual iteration: one 512-token chunk on top of what is cached and the running decodes.
        _attention("mistral_hybrid", "mistral-7b", "512@1871", 64, 256, 4096, lengths=4),
        # The model's sliding window, ragged chunk, contexts beyond the window.
        _attention("mistral_window", "mistral-7b", "435@6001", 77, 1024, 12288, lengths=5, window=4096),
        # Long contexts: three prompts in mid-prefill next to 128 decodes, 56 query heads.
        _attention("yi_long_hybrid", "yi-34b", "1024@9475,512@3210,384@11117", 128, 1024, 16384, lengths=6),
        # The largest batch: a thousand decodes and two chunks.
        _attention("llama70b_1024_decodes", "llama2-70b", "512@911,512@2840", 1024, 512, 4096, lengths=7),
        # Prefill alone, a 2048-token budget: a prompt's first tokens and the ragged rest of another's.
        _attention("llama70b_prefill", "llama2-70b", "1299@0,749@4211", 0, 0, 0),
        # Linear layers: a few decodes (weight fetch), a decode batch, the usual hybrid iteration, a large prefill budget.
        _linear("linear_mistral_8", "mistral-7b", 8),
        _linear("linear_yi_77", "yi-34b", 77),
        _linear("linear_mistral_576", "mistral-7b", 576),
        _linear("linear_llama70b_2048", "llama2-70b", 2048),
    ]


def _log_uniform(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def draw(rng):
    """One more case of the same ranges: batch sizes, contexts, chunk lengths and token counts over their logarithms."""
    if rng.random() < 0.4:
        c = _linear("", rng.choice(sorted(linear_layers.MODELS)), _log_uniform(rng, 1, 2048))
    else:
        heads = rng.choice(sorted(HEADS))
        mode = rng.choice(["decodes", "hybrid", "hybrid", "chunks"])
        high = _log_uniform(rng, 512, 16384)
        decodes = 0 if mode == "chunks" else max(1, min(_log_uniform(rng, 1, 1024), 2_000_000 // high))
        chunks = []
        if mode != "decodes":
            for _ in range(rng.choice([1, 1, 2, 3])):
                chunks.append("%d@%d" % (_log_uniform(rng, 17, 1024), rng.choice([0, _log_uniform(rng, 1, 12288)])))
        c = _attention("", heads, ",".join(chunks), decodes, _log_uniform(rng, 1, 256) if decodes else 0, high if decodes else 0,
                       rng.choice(["uniform", "lognormal"]), rng.randrange(1 << 20), rng.choice([0, 0, 0, 4096]),
                       rng.choice(["workspace", "workspace", "workspace", "noalloc"]))
    del c["name"]
    return c


def _lengths(case):
    """(q_len, ctx_len) of the batch: chunks first, then the decodes."""
    q_len, ctx = [], []
    for text in filter(None, case["chunks"].split(",")):
        new, prefix = (int(t) for t in text.split("@"))
        q_len.append(new)
        ctx.append(prefix + new)
    n, low, high = case["decodes"], case["low"], case["high"]
    rng = np.random.default_rng([case["lengths"], 0xCA5E])
    if case["spread"] == "lognormal":
        got = np.clip(np.rint(np.exp(math.log(max(1.0, high / 8)) + 0.8 * rng.standard_normal(n))), low, high)
    else:
        got = rng.integers(low, high + 1, size=n)
    return np.array(q_len + [1] * n, np.int32), np.array(ctx + [int(c) for c in got], np.int32)


def _prepare_attention(case, seed):
    hq, hkv, d = HEADS[case["heads"]]
    q_len, ctx_len = _lengths(case)
    tokens = int(q_len.sum())
    g = torch.Generator(device="cuda").manual_seed(seed)
    normal = lambda *shape: torch.randn(*shape, device="cuda", generator=g, dtype=torch.bfloat16)  # noqa: E731
    need = -(-ctx_len.astype(np.int64) // PAGE)
    pages = int(need.sum()) * 5 // 4 + 1   # a pool that is not full, pages of a sequence scattered over it
    order = torch.randperm(pages, device="cuda", generator=g, dtype=torch.int64).to(torch.int32)
    table = torch.full((len(q_len), int(need.max())), -1, device="cuda", dtype=torch.int32)
    at = 0
    for s, n in enumerate(need.tolist()):
        table[s, :n] = order[at:at + n]
        at += n
    handle = binding.Handle(hq, hkv, d, max_tokens=max(tokens, 4096), max_seqs=max(len(q_len), 64), max_blocks_per_seq=table.shape[1])
    if case["window"]:
        handle.set_option("window", case["window"])
    handle.ensure_workspace()
    q_start = np.concatenate([[0], np.cumsum(q_len)[:-1]]).astype(np.int32)
    return {"case": case, "handle": handle, "q_start": q_start, "q_len": q_len, "ctx_len": ctx_len, "table": table,
            "k_cache": normal(pages, hkv, PAGE, d), "v_cache": normal(pages, hkv, d, PAGE),
            "q": normal(tokens, hq, d), "k_new": normal(tokens, hkv, d), "v_new": normal(tokens, hkv, d),
            "out": torch.empty(tokens, hq, d, device="cuda", dtype=torch.bfloat16), "scale": 1.0 / math.sqrt(d)}


def _prepare_linear(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    layers, scratch = [], 16
    for _, n, k in linear_layers.layer_shapes(linear_layers.MODELS[case["model"]]):
        w = torch.randn(n, k, device="cuda", generator=g, dtype=torch.bfloat16) * (1.0 / math.sqrt(k))
        x = torch.randn(case["tokens"], k, device="cuda", generator=g, dtype=torch.bfloat16)
        layers.append((x, w, torch.empty(case["tokens"], n, device="cuda", dtype=torch.bfloat16)))
        scratch = max(scratch, binding.linear_workspace_bytes(case["tokens"], n, k))
    return {"case": case, "layers": layers, "scratch": torch.empty(scratch, device="cuda", dtype=torch.uint8)}


def prepare(case, seed):
    return _prepare_linear(case, seed) if case["kind"] == "linear" else _prepare_attention(case, seed)


def run(state):
    if state["case"]["kind"] == "linear":
        for x, w, y in state["layers"]:
            binding.linear(x, w, y, state["scratch"])
        return [y for _, _, y in state["layers"]]
    h, s = state["handle"], state
    h.kv_append(s["k_new"], s["v_new"], s["k_cache"], s["v_cache"], s["table"], s["q_start"], s["q_len"], s["ctx_len"])
    attend = h.hybrid_attention_noalloc if s["case"]["entry"] == "noalloc" else h.hybrid_attention
    out = attend(s["q"], s["k_cache"], s["v_cache"], s["table"], s["q_start"], s["q_len"], s["ctx_len"], s["scale"], s["out"])
    return {"out": out, "k_cache": s["k_cache"], "v_cache": s["v_cache"]}


def work(case):
    if case["kind"] == "linear":
        t = case["tokens"]
        shapes = linear_layers.layer_shapes(linear_layers.MODELS[case["model"]])
        return {"bytes": linear_layers.weight_bytes(shapes) + sum(2 * t * (n + k) for _, n, k in shapes),
                "flops": linear_layers.flops(shapes, t)}
    hq, hkv, d = HEADS[case["heads"]]
    cached = pairs = tokens = 0
    for q, c in zip(*(a.tolist() for a in _lengths(case))):
        w = case["window"] or c
        tokens += q
        cached += min(c - q, w - 1 if case["window"] else c)        # positions of earlier iterations that some row sees
        pairs += sum(min(p + 1, w) for p in range(c - q, c)) if case["window"] else q * (c - q) + q * (q + 1) // 2
    row = 2 * hkv * d * 2                                             # a position's key and value, all heads
    return {"bytes": cached * row + tokens * (2 * row + 2 * hq * d * 2), "flops": 4 * d * hq * pairs}


def tolerance(case):
    if case["kind"] == "linear":
        return {"rel": 7e-3}      # fp32 sums, one rounding to bf16: 1.7e-3 measured against 64 bits
    return {"rel": 9e-3}          # softmax weights rounded to bf16 as well: 2.0e-3 to 2.4e-3 measured against 64 bits


def exact(case, seed):
    s = prepare(case, seed)
    if case["kind"] == "linear":
        return [x.double() @ w.double().t().contiguous() for x, w, _ in s["layers"]]
    hq, hkv, d = HEADS[case["heads"]]
    group = hq // hkv
    out = torch.empty(s["out"].shape, device="cuda", dtype=torch.float64)
    for i, (t0, n, ctx) in enumerate(zip(s["q_start"].tolist(), s["q_len"].tolist(), s["ctx_len"].tolist())):
        own = s["table"][i, : -(-ctx // PAGE)].long()
        k = s["k_cache"][own].permute(0, 2, 1, 3).reshape(-1, hkv, d)[:ctx].double()
        v = s["v_cache"][own].permute(0, 3, 1, 2).reshape(-1, hkv, d)[:ctx].double()
        k[ctx - n:] = s["k_new"][t0:t0 + n].double()
        v[ctx - n:] = s["v_new"][t0:t0 + n].double()
        k, v = k.permute(1, 2, 0).contiguous(), v.permute(1, 0, 2).contiguous()     # [Hkv, d, ctx], [Hkv, ctx, d]
        keys = torch.arange(ctx, device="cuda")
        for r0 in range(0, n, 256):
            r1 = min(n, r0 + 256)
            at = torch.arange(ctx - n + r0, ctx - n + r1, device="cuda")
            q = s["q"][t0 + r0:t0 + r1].double().reshape(r1 - r0, hkv, group, d).permute(1, 0, 2, 3).reshape(hkv, -1, d).contiguous()
            scores = torch.bmm(q, k).reshape(hkv, r1 - r0, group, ctx) * s["scale"]
            seen = keys[None, :] <= at[:, None]
            if case["window"]:
                seen &= keys[None, :] > at[:, None] - case["window"]
            p = torch.softmax(scores.masked_fill_(~seen[None, :, None, :], -math.inf), dim=-1)
            o = torch.bmm(p.reshape(hkv, -1, ctx), v).reshape(hkv, r1 - r0, group, d)
            out[t0 + r0:t0 + r1] = o.permute(1, 0, 2, 3).reshape(r1 - r0, hq, d)
    return {"out": out, "k_cache": None, "v_cache": None}
