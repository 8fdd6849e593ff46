"""Timed cases of the KV-cache path: what a serving program has the library do, through its public calls.

Shapes are those of the workloads in kvq_workloads.py (Llama-3.1-8B: 32 query heads / 8 kv heads, keys with three
channels x10; Qwen2.5-7B: 28 / 4, keys with a per-channel offset of standard deviation 20) and of the small grouped-query
test configuration (8 / 2), head dimension 128, with the layer-wise precision pairs of their schedules.  A case covers a
few layers in the schedule's proportions, not all 28 or 32, so that inputs are made quickly; the caches of the large ones
are several times the last-level cache all the same.

Kinds of case (`kind`):
  decode    one decode step's attention over filled caches, layer by layer (what a step costs when the model appends
            through kvq_quantize_append or attends to a cache as it stands)
  generate  a prompt quantized into every layer, then `steps` fused append-and-attend steps per layer, window flushes
            included (one request batch from its prompt to its last token)
  ingest    a prompt quantized into every layer, then the first token's attention (time to first token of a program
            whose prompt attention reads the unquantized keys and values)
  prefill   a prompt quantized into every layer, then the prompt's own causal attention over the quantized cache
  chunk     causal attention of the last `n_q` tokens over a long filled cache (chunked prefill, verification of drafts)
"""
import math

import torch

from paper_2502_04420_amd import KVQ

D, G = 128, 32
SHAPES = {"llama8b": (32, 8), "qwen7b": (28, 4), "gqa8x2": (8, 2)}
KINDS = ("decode", "generate", "ingest", "prefill", "chunk")


def _case(name, kind, shape, batch, context, pairs, n_q=0, steps=0, residual=32, meta16=False, per_token=False, noalloc=False):
    return {"name": name, "kind": kind, "shape": shape, "batch": batch, "context": context, "pairs": pairs, "n_q": n_q,
            "steps": steps, "residual": residual, "meta16": meta16, "per_token": per_token, "noalloc": noalloc}


def listed():
    return [
        # the smallest call there is in earnest: one layer of the small grouped-query model, one sequence
        _case("decode_tiny", "decode", "gqa8x2", 1, 512, "K8V4", noalloc=True),
        # one chat: a single sequence, every layer of a step has little to read; ragged length, searched 3.25-bit pairs
        _case("decode_chat", "decode", "llama8b", 1, 4133, "K8V4,K4V4,K4V4" + ",K4V2" * 11 + ",K2V2,K2V2"),
        # the benchmark's batch: 3.25-bit mix (a quarter of the layers K4V4, the others K4V2)
        _case("decode_batch", "decode", "llama8b", 16, 8192, "K4V4,K4V4" + ",K4V2" * 6),
        # long contexts at a full batch: the largest caches
        _case("decode_long", "decode", "llama8b", 32, 32768, "K4V4,K4V2,K4V2,K4V2"),
        # seven query heads per kv head, keys with an offset on every channel, 4.0-bit mix
        _case("decode_qwen", "decode", "qwen7b", 8, 32768, "K8V2,K4V2,K8V2,K4V2"),
        # the two baselines a quantized cache is held against: uniform 8 bits, and half precision at an odd length
        _case("decode_kv8", "decode", "llama8b", 16, 4096, "K8V8,K8V8,K8V8,K8V8"),
        _case("decode_half", "decode", "llama8b", 8, 4519, "K16V16,K16V16,K16V16,K16V16"),
        # a small batch from prompt to last token: searched 4.90-bit pairs, the other key grouping and scale precision
        _case("generate", "generate", "llama8b", 4, 733, "K8V4,K8V4,K8V4,K4V4,K4V2,K2V2", steps=48, meta16=True, per_token=True),
        # quantize-and-pack of a large batch of prompts, then the first token
        _case("ingest", "ingest", "llama8b", 16, 8192, "K4V4,K4V2"),
        # one user's prompt of ordinary, odd length
        _case("prefill_chat", "prefill", "llama8b", 1, 2027, "K4V4,K4V2,K4V2,K2V2"),
        # a batch of long prompts
        _case("prefill_batch", "prefill", "llama8b", 4, 8192, "K4V2"),
        # the last chunk of a long prompt that is taken 512 tokens at a time
        _case("chunk_long", "chunk", "llama8b", 1, 24576, "K4V4,K4V2,K4V2,K2V2", n_q=512),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case.  Every kind keeps below the largest listed one (the caches of decode_long, the attention of
    prefill_batch) by bounding batch x context, the number of layers and the number of query-token pairs."""
    kind = rng.choice(KINDS + ("decode", "decode", "prefill", "chunk"))
    shape = rng.choice(("llama8b", "llama8b", "qwen7b", "gqa8x2"))
    hq, hkv = SHAPES[shape]
    bits = {"searched": ("K8V4", "K4V4", "K4V2", "K2V2"), "wide": ("K8V8", "K8V4", "K8V2"), "narrow": ("K4V4", "K4V2", "K2V2", "K2V4"),
            "half": ("K16V16", "K8V8")}[rng.choice(("searched", "searched", "narrow", "narrow", "wide", "half"))]
    layers = rng.randint(1, 4)
    pairs = ",".join(rng.choice(bits) for _ in range(layers))
    options = dict(residual=rng.choice((32, 32, 32, 0, 64, 128)), meta16=rng.random() < 0.3, per_token=rng.random() < 0.25)
    if kind == "decode":
        context = _log_uniform(rng, 33, 32768)
        batch = _log_uniform(rng, 1, max(1, min(64, 8 * 16 * 32768 // (context * hkv * layers))))
        return _strip(_case("", kind, shape, batch, context, pairs, noalloc=rng.random() < 0.25, **options))
    if kind == "generate":
        context, steps = _log_uniform(rng, 1, 4096), rng.randint(8, 64)
        return _strip(_case("", kind, shape, _log_uniform(rng, 1, 16), context, pairs, steps=steps, **options))
    if kind == "ingest":
        context = _log_uniform(rng, 33, 16384)
        batch = _log_uniform(rng, 1, max(1, min(64, 8 * 16 * 8192 // (context * hkv))))
        return _strip(_case("", kind, shape, batch, context, pairs, **options))
    if kind == "prefill":
        # at most two thirds of prefill_batch's 4 x 32 x 8192^2 / 2 query-token pairs over all layers
        context = _log_uniform(rng, 17, 8192)
        batch = _log_uniform(rng, 1, max(1, min(32, int(2.6 * 32 * 8192 ** 2 / (hq * context ** 2 * layers)))))
        while layers > 1 and batch * hq * context ** 2 * layers > 2.7 * 32 * 8192 ** 2:
            layers -= 1
        return _strip(_case("", kind, shape, batch, context, ",".join(pairs.split(",")[:layers]), **options))
    context = _log_uniform(rng, 2048, 32768)
    n_q = _log_uniform(rng, 8, 1024)
    return _strip(_case("", kind, shape, rng.choice((1, 1, 2, 4)), context, pairs, n_q=n_q, **options))


def _strip(case):
    case = dict(case)
    del case["name"]
    return case


# ------------------------------------------------------------------ inputs


def _pairs(case):
    out = []
    for item in case["pairs"].split(","):
        k, v = item[1:].split("V")
        out.append((int(k), int(v)))
    return out


def _generator(seed, layer):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1009 + 17 * layer + 5)
    return g


def _tokens(case, seed, layer, n, extra=0):
    """fp16 keys and values [B, Hkv, n, D] of one layer on the GPU, and its fp16 queries [B, Hq, extra, D]."""
    hq, hkv = SHAPES[case["shape"]]
    g = _generator(seed, layer)
    shape = (case["batch"], hkv, n, D)
    scale = torch.ones(hkv, 1, D, device="cuda", dtype=torch.float16)
    offset = torch.zeros(hkv, 1, D, device="cuda", dtype=torch.float16)
    if case["shape"] == "qwen7b":
        offset = (20.0 * torch.randn(hkv, 1, D, generator=g, device="cuda")).to(torch.float16)
    else:
        large = torch.rand(hkv, D, generator=g, device="cuda").topk(3, dim=1).indices
        scale.view(hkv, D).scatter_(1, large, 10.0)
    q = torch.randn((case["batch"], hq, extra, D), generator=g, device="cuda", dtype=torch.float16) if extra else None
    K = torch.randn(shape, generator=g, device="cuda", dtype=torch.float16)
    K.mul_(scale).add_(offset)
    V = torch.randn(shape, generator=g, device="cuda", dtype=torch.float16)
    return K, V, q


def _n_queries(case):
    """Query positions per layer and pass."""
    return {"decode": 1, "ingest": 1, "generate": case["steps"], "prefill": case["context"], "chunk": min(case["n_q"], case["context"])}[case["kind"]]


def _total(case):
    return case["context"] + (case["steps"] if case["kind"] == "generate" else 0)


def prepare(case, seed):
    hq, hkv = SHAPES[case["shape"]]
    pairs, B, nq = _pairs(case), case["batch"], _n_queries(case)
    kind = case["kind"]
    cache = KVQ(len(pairs), B, hq, hkv, D, _total(case), [p[0] for p in pairs], [p[1] for p in pairs], residual=case["residual"],
                meta_dtype=int(case["meta16"]), key_mode=int(case["per_token"]))
    state = {"cache": cache, "kind": kind, "layers": []}
    for layer in range(len(pairs)):
        K, V, q = _tokens(case, seed, layer, _total(case), nq)
        entry = {"layer": layer}
        if kind in ("decode", "chunk"):
            cache.quantize_append(layer, K, V)                    # the cache is what such a program has in hand
        else:
            T = case["context"]
            entry["prompt"] = (K[:, :, :T].contiguous(), V[:, :, :T].contiguous())
        if kind in ("prefill", "chunk"):
            entry["q"] = q
            entry["out"] = torch.empty_like(q)
        elif kind == "generate":
            entry["steps"] = []
            entry["outs"] = torch.empty((case["steps"], B, hq, D), dtype=torch.float16, device="cuda")
            for s in range(case["steps"]):
                t = case["context"] + s
                entry["steps"].append((K[:, :, t:t + 1].contiguous(), V[:, :, t:t + 1].contiguous(), q[:, :, s].contiguous(), entry["outs"][s]))
        else:
            entry["q"] = q[:, :, 0].contiguous()
            entry["out"] = torch.empty_like(entry["q"])
        state["layers"].append(entry)
    state["attend"] = cache.decode_attention_noalloc if case["noalloc"] else cache.decode_attention
    state["outputs"] = [e["outs"] if kind == "generate" else e["out"] for e in state["layers"]]
    return state


def run(state):
    cache, layers, kind = state["cache"], state["layers"], state["kind"]
    if kind == "decode":
        attend = state["attend"]
        for e in layers:
            attend(e["layer"], e["q"], e["out"])
    elif kind == "chunk":
        for e in layers:
            cache.prefill_attention(e["layer"], e["q"], e["out"])
    else:
        cache.reset()
        for e in layers:
            cache.quantize_append(e["layer"], *e["prompt"])
            if kind == "ingest":
                cache.decode_attention(e["layer"], e["q"], e["out"])
            elif kind == "prefill":
                cache.prefill_attention(e["layer"], e["q"], e["out"])
        if kind == "generate":
            for step in zip(*(e["steps"] for e in layers)):
                for layer, (k, v, q, out) in enumerate(step):
                    cache.append_decode_attention(layer, k, v, q, out)
    return state["outputs"]


# ------------------------------------------------------------------ what a pass cannot do without


def _packed(T, residual):
    return G * (max(T - residual, 0) // G)


def _token_bytes(bits, meta16):
    """Bytes of one quantized token of one head: codes, then four (scale, zero-point) pairs (fp16 zero-points)."""
    return D * bits // 8 + (0 if bits == 16 else 4 * ((2 if meta16 else 4) + 2))


def _cache_bytes(case, pair, T):
    """All bytes one layer holds for T tokens."""
    heads = case["batch"] * SHAPES[case["shape"]][1]
    n_p = _packed(T, case["residual"])
    return heads * (n_p * (_token_bytes(pair[0], case["meta16"]) + _token_bytes(pair[1], case["meta16"])) + (T - n_p) * 4 * D)


def work(case):
    hq, hkv = SHAPES[case["shape"]]
    B, T, kind, nq = case["batch"], case["context"], case["kind"], _n_queries(case)
    bytes_, flops = 0.0, 0.0
    for pair in _pairs(case):
        if kind == "generate":
            for s in range(case["steps"]):
                bytes_ += _cache_bytes(case, pair, T + s + 1)
                flops += 4.0 * D * B * hq * (T + s + 1)
        else:
            bytes_ += _cache_bytes(case, pair, T)
            flops += 4.0 * D * B * hq * (nq * T - nq * (nq - 1) // 2)
        bytes_ += 2 * B * hq * nq * D * 2                            # queries read, outputs written
        if kind in ("generate", "ingest", "prefill"):
            bytes_ += 2 * B * hkv * _total(case) * D * 2             # keys and values read ...
            bytes_ += _cache_bytes(case, pair, _total(case))         # ... and stored
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    # 2-norm against 64 bits, measured over the listed cases: 2.0e-4 (the fp16 rounding of the outputs alone) to 4.8e-4 for
    # decode steps, 3.0e-4 .. 3.5e-4 for prefill-stage attention, which also rounds the softmax weights and the dequantized
    # operands to fp16.  About four times that.
    # "max": largest difference in units of the outputs' root mean square, or of the value itself where that is larger.
    if case["kind"] in ("prefill", "chunk"):
        return {"rel": 1.5e-3, "max": 3e-2}
    return {"rel": 1.5e-3, "max": 1e-2}


# ------------------------------------------------------------------ the same in 64 bits, plain torch


def _dequantized(x, bits, meta16, per_token):
    """x: fp16 [n, D] with n a multiple of 32.  Eq. 2 per group of 32 tokens (per channel) or of 32 channels (per token)."""
    if bits == 16:
        return x.double()
    g = x.double().view(-1, D // G, G) if per_token else x.double().view(-1, G, D)
    dim = 2 if per_token else 1
    z = g.amin(dim, keepdim=True)
    s = ((g.amax(dim, keepdim=True) - z).float().double() / (2 ** bits - 1)).float()  # the stored scale: fp32, or rounded once more to fp16
    s = (s.half() if meta16 else s).double()
    # The codes are whole numbers that the format fixes to the bit: fp32 difference, fp32 quotient (the 64-bit one rounded
    # once more is the same), round half to even.  In 64 bits throughout, quotients next to a tie would get other codes.
    d = g.float().sub_(z.float()).double()
    codes = torch.round(torch.where(s > 0, d / torch.where(s > 0, s, torch.ones_like(s)), torch.zeros_like(d)).float()).double()
    return (codes.clamp_(0, 2 ** bits - 1).mul_(s).add_(z)).view(-1, D)


def _head_attention(case, pair, K, V, q, T):
    """One (sequence, kv head): fp16 K, V [>= T, D], q [g, n, D] = the last n of T positions (n = 1: no mask needed)."""
    n_p = _packed(T, case["residual"])
    Kd = torch.cat((_dequantized(K[:n_p], pair[0], case["meta16"], case["per_token"]), K[n_p:T].double()))
    Vd = torch.cat((_dequantized(V[:n_p], pair[1], case["meta16"], True), V[n_p:T].double()))
    n = q.shape[1]
    out = torch.empty(q.shape, dtype=torch.float64, device=q.device)
    pos = torch.arange(T - n, T, device=q.device)
    keys = torch.arange(T, device=q.device)
    for j in range(q.shape[0]):
        for i in range(0, n, 4096):
            p = pos[i:i + 4096]
            top = int(p[-1]) + 1
            s = torch.mm(q[j, i:i + 4096].double(), Kd[:top].t().contiguous()).mul_(1.0 / math.sqrt(D))
            if n > 1:
                s.masked_fill_(keys[None, :top] > p[:, None], -math.inf)
            out[j, i:i + 4096] = torch.mm(torch.softmax(s, dim=1), Vd[:top])
    return out


def exact(case, seed):
    if case["batch"] * SHAPES[case["shape"]][1] * len(_pairs(case)) * max(1, case["steps"]) > 20000:
        return None                                                  # many tiny heads: minutes of launches
    hq, hkv = SHAPES[case["shape"]]
    gq, outs = hq // hkv, []
    for layer, pair in enumerate(_pairs(case)):
        K, V, q = _tokens(case, seed, layer, _total(case), _n_queries(case))
        out = torch.empty(q.shape, dtype=torch.float64, device="cuda")
        for b in range(case["batch"]):
            for h in range(hkv):
                qh = q[b, h * gq:(h + 1) * gq]
                if case["kind"] == "generate":
                    for s in range(case["steps"]):
                        out[b, h * gq:(h + 1) * gq, s:s + 1] = _head_attention(case, pair, K[b, h], V[b, h], qh[:, s:s + 1], case["context"] + s + 1)
                else:
                    out[b, h * gq:(h + 1) * gq] = _head_attention(case, pair, K[b, h], V[b, h], qh, case["context"])
        if case["kind"] == "generate":
            outs.append(out.permute(2, 0, 1, 3).contiguous())
        else:
            outs.append(out if case["kind"] in ("prefill", "chunk") else out[:, :, 0].contiguous())
    return outs
