"""Workloads that the speed of this library is measured on, through its public entry points.

A program that uses the library does two things with it: it prefills prompts (`pop_prefill`, the pruned
prefill with the boundary token and its logits) and it decodes (`pop_decode_step`, one token per sequence
against the paged cache).  The cases below are those two calls over the model shapes of
`paper_2602_03295_amd.synth` (Llama-3.1-8B, Qwen3-VL-8B-style, Gemma-3-12B-style, the tiny fp32 model), from
a handful of rows to 32768 tokens.  Every layer is as wide as the real model's; the depth is cut to four layers
(six where five sliding-window layers precede a global one) and the vocabulary by the same ratio, so that the
LM head keeps its share of a call and a state fits the card several times.  The weights of such a stack are
still larger than any cache of the chip: they come from HBM in every pass, as in the full model.

`exact` computes the same outputs in 64 bits with plain torch from the inputs alone.
"""
import math

import numpy as np
import torch

from paper_2602_03295_amd import pop, synth

PAGE = 16
DECODE_ROOM = 1024          # positions a decode case can advance before its sequences are started anew
# shape -> (layers, layers of the full model)
DEPTH = {"llama8b": (4, 32), "qwen3vl8b": (4, 36), "gemma12b": (6, 48), "tiny": (8, 8)}


def _prefill(name, shape, lens, l_keep, **kw):
    return _case(name, kind="prefill", shape=shape, lens=lens, l_keep=l_keep, **kw)


def _decode(name, shape, lens, **kw):
    return _case(name, kind="decode", shape=shape, lens=lens, l_keep=0, **kw)


def _case(name, lens, **kw):
    case = {"lens": ",".join(map(str, lens)), "fp32": False, "fp8": False, "qk_norm": False, "visual": 0, **kw}
    return case if name is None else {"name": name, **case}


def listed():
    return [
        # the small fp32 model that numerical checks of a port are made on: one 128-token prompt, launches count
        _prefill("tiny_fp32_128", "tiny", [128], 5, fp32=True),
        # a batch of one-line questions: time to first token is weight streaming
        _prefill("llama_8x32", "llama8b", [32] * 8, 3),
        # a few short chat turns of unequal, odd length arriving together
        _prefill("llama_short_ragged", "llama8b", [77, 301, 150], 3),
        # the headline workload: one 2048-token prompt
        _prefill("llama_2k", "llama8b", [2048], 3),
        # a serving batch: eight prompts of 512 to 4096 tokens
        _prefill("llama_ragged_20k", "llama8b", [1427, 3804, 2613, 3898, 660, 2279, 4069, 1111], 3),
        # an image and a question: 4096 supplied rows inside a 6144-token prompt
        _prefill("qwen_visual_6k", "qwen3vl8b", [6144], 3, visual=4096),
        # sliding-window layers with wide heads on a long document
        _prefill("gemma_16k", "gemma12b", [16384], 4),
        # the longest prompt
        _prefill("llama_32k", "llama8b", [32768], 3),
        # decoding for one user
        _decode("decode_1x2k", "llama8b", [2048]),
        # decoding for a small batch
        _decode("decode_8x2k", "llama8b", [2048, 1979, 2048, 1500, 2048, 2021, 1777, 2048]),
        # long contexts, where the 8-bit cache is chosen to fit them
        _decode("decode_8x8k_fp8", "llama8b", [8192, 8000, 8192, 7777, 8192, 8192, 8100, 8192], fp8=True),
        # a busy server: 32 sequences of about 512 tokens
        _decode("decode_32x512", "qwen3vl8b", [512 - 7 * (i % 5) for i in range(32)]),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _split(rng, total, n):
    """n unequal positive lengths that add up to about `total`."""
    w = [rng.uniform(0.3, 1.0) for _ in range(n)]
    return [max(1, int(total * x / sum(w))) for x in w]


def draw(rng):
    shape = rng.choice(["llama8b", "llama8b", "qwen3vl8b", "gemma12b"])
    kind = rng.choice(["prefill", "prefill", "prefill", "prefill", "decode", "decode", "decode", "decode", "fp32"])
    if kind == "fp32":
        # one or several small prompts on the fp32 model, up to a thousand tokens
        total = _log_int(rng, 24, 1000)
        n = rng.choice([1, 1, 2, 5])
        return _prefill(None, "tiny", _split(rng, total, n), rng.randint(3, 8), fp32=True)
    n_layers = DEPTH[shape][0]
    if kind == "prefill":
        # most prompts are pruned by a quarter to a third; some programs run the full depth
        l_keep = rng.choice([n_layers - 1, n_layers - 1, n_layers - 2, n_layers])
        total = _log_int(rng, 24, 16000 if shape == "gemma12b" else (20000 if l_keep == n_layers else 30000))
        n = rng.choice([1, 1, 1, 2, 3, 5, 8]) if total >= 64 else 1
        return _prefill(None, shape, _split(rng, total, n), l_keep, qk_norm=shape != "llama8b" and rng.random() < 0.5,
                        visual=0 if shape != "qwen3vl8b" or n > 1 else total // 2)
    n = _log_int(rng, 1, 48)
    context = _log_int(rng, 60, min(16000, 60000 // n))
    lens = [max(1, context - rng.randint(0, context // 4)) for _ in range(n)]
    return _decode(None, shape, lens, fp8=rng.random() < 0.3, qk_norm=shape != "llama8b" and rng.random() < 0.5)


# --------------------------------------------------------------------------------------------- inputs
def _lens(case):
    return [int(x) for x in case["lens"].split(",")]


def _config(case):
    n_layers, full = DEPTH[case["shape"]]
    cfg = synth.get_config(case["shape"])
    cfg.update(n_layers=n_layers, vocab=cfg["vocab"] * n_layers // full // 32 * 32 if full != n_layers else cfg["vocab"],
               dtype=pop.DTYPE_F32 if case["fp32"] else pop.DTYPE_BF16,
               kv_dtype=pop.KV_FP8_E4M3 if case["fp8"] else pop.KV_BF16)
    if case["fp8"]:
        cfg.update(k_scale=0.03, v_scale=0.02)
    return cfg


def _weights(cfg, case, gen):
    """Random weights in the layout the library takes (wqkv rows q | k | v, w_gate_up rows gate | up)."""
    d, hd, f, v = cfg["d_model"], cfg["head_dim"], cfg["d_ffn"], cfg["vocab"]
    dq, dkv = cfg["n_q_heads"] * hd, cfg["n_kv_heads"] * hd
    dt = torch.float32 if case["fp32"] else torch.bfloat16

    def matrix(*shape):
        return torch.empty(*shape, dtype=dt, device="cuda").normal_(0.0, 0.02, generator=gen)

    def scale(n):
        return torch.empty(n, dtype=torch.float32, device="cuda").normal_(1.0, 0.1, generator=gen)

    w = {"embed": matrix(v, d), "lm_head": matrix(v, d), "final_norm": scale(d), "layers": []}
    for _ in range(cfg["n_layers"]):
        lw = {"norm_in": scale(d), "wqkv": matrix(dq + 2 * dkv, d), "wo": matrix(d, dq), "norm_post": scale(d),
              "w_gate_up": matrix(2 * f, d), "w_down": matrix(d, f)}
        if case["qk_norm"]:
            lw.update(q_norm=scale(hd), k_norm=scale(hd))
        w["layers"].append(lw)
    return w


def _inputs(case, seed):
    """Everything that is drawn: (config, weights, host tokens, visual rows, host block table, pages, cache values)."""
    cfg, lens = _config(case), _lens(case)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    host = np.random.RandomState(seed % (1 << 31))
    w = _weights(cfg, case, gen)
    decode = case["kind"] == "decode"
    tokens = host.randint(0, cfg["vocab"], size=sum(lens)).astype(np.int32)
    # pages in no particular order, as a server's free list hands them out
    per = [(n + (DECODE_ROOM if decode else 0) + PAGE - 1) // PAGE for n in lens]
    ids = host.permutation(sum(per)).astype(np.int32)
    table = np.full((len(lens), max(per)), -1, dtype=np.int32)
    at = 0
    for b, n in enumerate(per):
        table[b, :n] = ids[at:at + n]
        at += n
    visual = None
    if case["visual"]:
        visual = torch.empty(case["visual"], cfg["d_model"], device="cuda").normal_(0.0, 1.0, generator=gen).to(torch.bfloat16)
    entries = None
    if decode:
        # what earlier calls have left in the cache, at the spread that LN(x) W^T has with these weights
        std = 0.02 * math.sqrt(cfg["d_model"])
        shape = (cfg["n_layers"], 2, sum(per), cfg["n_kv_heads"], PAGE, cfg["head_dim"])
        entries = torch.empty(shape, dtype=torch.float32 if case["fp32"] else torch.bfloat16, device="cuda")
        entries.normal_(0.0, std, generator=gen)
        if case["fp8"]:
            codes = torch.empty(shape, dtype=torch.uint8, device="cuda")
            for l in range(shape[0]):
                for kv, s in ((0, cfg["k_scale"]), (1, cfg["v_scale"])):
                    codes[l, kv] = (entries[l, kv].float() / s).clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
            entries = codes
    step_tokens = host.randint(0, cfg["vocab"], size=(DECODE_ROOM, len(lens))).astype(np.int32)
    return cfg, w, tokens, visual, table, sum(per), entries, step_tokens


def _start_sequences(s):
    """The prompts of a decode case enter the cache (the body alone, no layer kept)."""
    pop.pop_prefill(s["model"], s["cache"], s["tokens"], s["cu"], s["table"], 0, s["prefill_workspace"],
                    mode=pop.MODE_BODY_ONLY)


def prepare(case, seed):
    cfg, w, tokens, visual, table, n_pages, entries, step_tokens = _inputs(case, seed)
    lens = _lens(case)
    n = len(lens)
    model = pop.Model(cfg, w)
    cache = pop.Cache(cfg, n_pages, n, table.shape[1], fill=0.0)
    s = {"case": case, "model": model, "cache": cache, "tokens": tokens, "table": table,
         "cu": np.concatenate([[0], np.cumsum(lens)]).astype(np.int32),
         "logits": torch.empty(n, cfg["vocab"], dtype=torch.float32, device="cuda")}
    s["prefill_workspace"] = pop.alloc_workspace(cfg, sum(lens), n, table.shape[1])
    # the pool as a tensor of numbers (an 8-bit cache: its codes)
    s["pool"] = cache.pool.view(torch.float8_e4m3fn) if cache.fp8 else cache.pool
    if case["kind"] == "prefill":
        s["visual"] = visual
        s["ranges"] = None if visual is None else [[0, 64 if 64 + len(visual) <= lens[0] else 0, len(visual)]]
    else:
        s["workspace"] = pop.alloc_workspace(cfg, n, n, table.shape[1])
        s["step_tokens"], s["step"] = step_tokens, 0
        _start_sequences(s)
        cache.pool.copy_(entries.view(-1))
    return s


def run(s):
    case = s["case"]
    if case["kind"] == "prefill":
        pop.pop_prefill(s["model"], s["cache"], s["tokens"], s["cu"], s["table"], case["l_keep"], s["prefill_workspace"],
                        logits=s["logits"], embeds=s["visual"], embed_ranges=s["ranges"])
    else:
        if s["step"] == DECODE_ROOM:        # the sequences are full: the next ones take their place
            _start_sequences(s)
            s["step"] = 0
        pop.pop_decode_step(s["model"], s["cache"], s["step_tokens"][s["step"]], s["workspace"], logits=s["logits"])
        s["step"] += 1
    return {"logits": s["logits"], "pool": s["pool"]}


# --------------------------------------------------------------------------------------------- what a pass costs
def _is_global(cfg, layer):
    return cfg["sliding_window"] == 0 or cfg["global_every"] == 0 or (layer + 1) % cfg["global_every"] == 0


def work(case):
    cfg, lens = _config(case), _lens(case)
    d, hd, f, v, n_layers = cfg["d_model"], cfg["head_dim"], cfg["d_ffn"], cfg["vocab"], cfg["n_layers"]
    dq, dkv = cfg["n_q_heads"] * hd, cfg["n_kv_heads"] * hd
    esz = 4 if case["fp32"] else 2
    kv_esz = 4 if case["fp32"] else (1 if case["fp8"] else 2)
    full = (dq + 2 * dkv) * d + d * dq + 3 * d * f       # weights of a layer
    rows, n = sum(lens), len(lens)
    weights = v * d + n_layers * full                    # LM head and every layer: the last token runs all of them
    flops, cache = 2.0 * n * v * d, 0.0

    def keys(length, layer):     # (query, key) pairs of one causal pass
        w = length if _is_global(cfg, layer) else min(length, cfg["sliding_window"])
        return w * (w + 1) / 2.0 + (length - w) * float(w)

    for layer in range(n_layers):
        if case["kind"] == "decode":
            seen = sum((m + 1) if _is_global(cfg, layer) else min(m + 1, cfg["sliding_window"]) for m in lens)
            flops += 2.0 * n * full + 4.0 * dq * seen
            cache += 2.0 * dkv * kv_esz * seen
        elif layer < case["l_keep"]:
            flops += 2.0 * rows * full + sum(4.0 * dq * keys(m, layer) for m in lens)
            cache += 2.0 * dkv * kv_esz * rows
        else:
            seen = sum(m if _is_global(cfg, layer) else min(m, cfg["sliding_window"]) for m in lens)
            flops += 2.0 * rows * 2 * dkv * d + 2.0 * n * full + 4.0 * dq * seen
            cache += 2.0 * dkv * kv_esz * (rows + seen)
    fed = n if case["kind"] == "decode" else rows
    return {"bytes": weights * float(esz) + cache + fed * d * float(esz) + 4.0 * n * v, "flops": flops}


def tolerance(case):
    if case["fp32"]:
        return {"rel": 1e-5}
    # bf16 inputs of every projection: a changed order of sums moves roundings that travel through the layers
    return {"rel": 2e-2}


# --------------------------------------------------------------------------------------------- 64 bits
def _norm(x, gamma, eps):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + eps) * gamma.double()


def _rope(x, pos, theta):
    """x [rows, heads, hd], pairs (i, i + hd/2)."""
    half = x.shape[-1] // 2
    i = torch.arange(half, dtype=torch.float64, device=x.device)
    ang = pos.double()[:, None] * theta ** (-2.0 * i / x.shape[-1])
    c, s = torch.cos(ang)[:, None, :], torch.sin(ang)[:, None, :]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], dim=-1)


def _qkv(cfg, lw, layer, x, pos):
    hd, hq, hkv = cfg["head_dim"], cfg["n_q_heads"], cfg["n_kv_heads"]
    y = _norm(x, lw["norm_in"], cfg["rms_eps"]) @ lw["wqkv"].double().t()
    q, k, v = y.split([hq * hd, hkv * hd, hkv * hd], dim=1)
    q, k, v = q.reshape(-1, hq, hd), k.reshape(-1, hkv, hd), v.reshape(-1, hkv, hd)
    if "q_norm" in lw:
        q, k = _norm(q, lw["q_norm"], cfg["rms_eps"]), _norm(k, lw["k_norm"], cfg["rms_eps"])
    theta = cfg["rope_theta"] if _is_global(cfg, layer) else cfg["rope_theta_local"]
    return _rope(q, pos, theta), _rope(k, pos, theta), v


def _attend(cfg, layer, q, qpos, k, v):
    """q [rows, hq, hd] at positions qpos over k, v [positions, hkv, hd]; blocks of rows bound the memory."""
    hd, g = cfg["head_dim"], cfg["n_q_heads"] // cfg["n_kv_heads"]
    window = 0 if _is_global(cfg, layer) else cfg["sliding_window"]
    out = torch.empty_like(q)
    first = int(qpos[0])
    for r0 in range(0, len(qpos), 2048):
        r1 = min(r0 + 2048, len(qpos))
        lo = max(0, first + r0 - window + 1) if window else 0
        hi = first + r1
        p = torch.arange(lo, hi, device=q.device)
        hidden = p[None, :] > qpos[r0:r1, None]
        if window:
            hidden = hidden | (p[None, :] <= qpos[r0:r1, None] - window)
        for h in range(cfg["n_q_heads"]):
            s = (q[r0:r1, h] @ k[lo:hi, h // g].t().contiguous()) / math.sqrt(hd)
            s.masked_fill_(hidden, -math.inf)
            out[r0:r1, h] = torch.softmax(s, dim=-1) @ v[lo:hi, h // g].contiguous()
    return out.reshape(len(qpos), -1)


def _finish_layer(cfg, lw, x, attn):
    x = x + attn @ lw["wo"].double().t()
    m = _norm(x, lw["norm_post"], cfg["rms_eps"])
    f = cfg["d_ffn"]
    gate = m @ lw["w_gate_up"][:f].double().t()
    act = torch.nn.functional.silu(gate) if cfg["act"] == synth.ACT_SILU else torch.nn.functional.gelu(gate, approximate="tanh")
    del gate
    act *= m @ lw["w_gate_up"][f:].double().t()
    return x + act @ lw["w_down"].double().t()


def _logits(cfg, w, x):
    return _norm(x, w["final_norm"], cfg["rms_eps"]) @ w["lm_head"].double().t()


def _stored(cfg, x, kv):
    """What attention reads of a new entry: with the 8-bit cache, the value of the code it is stored as."""
    if cfg["kv_dtype"] != pop.KV_FP8_E4M3:
        return x
    s = cfg["k_scale"] if kv == 0 else cfg["v_scale"]
    return (x / s).float().clamp(-448, 448).to(torch.float8_e4m3fn).double() * s


def exact(case, seed):
    cfg, w, tokens, visual, table, n_pages, entries, step_tokens = _inputs(case, seed)
    lens = _lens(case)
    starts = np.concatenate([[0], np.cumsum(lens)])
    hkv, hd = cfg["n_kv_heads"], cfg["head_dim"]
    dev = w["embed"].device
    scales = (cfg["k_scale"], cfg["v_scale"]) if case["fp8"] else (1.0, 1.0)
    if entries is None:
        pool = torch.zeros(cfg["n_layers"], 2, n_pages, hkv, PAGE, hd, dtype=torch.float64, device=dev)
    elif case["fp8"]:
        pool = entries.view(torch.float8_e4m3fn).to(torch.float64)
    else:
        pool = entries.double()

    def places(b, n):
        t = torch.arange(n, device=dev)
        return torch.as_tensor(table[b], device=dev).long()[t // PAGE], t % PAGE

    if case["kind"] == "decode":
        x = w["embed"][torch.as_tensor(step_tokens[0], device=dev).long()].double()
        pos = torch.as_tensor(lens, device=dev)
        for layer, lw in enumerate(w["layers"]):
            q, k, v = _qkv(cfg, lw, layer, x, pos)
            out = []
            for b, n in enumerate(lens):
                page, off = places(b, n + 1)
                for kv, new in ((0, k), (1, v)):
                    pool[layer, kv, page[n], :, off[n]] = _stored(cfg, new[b], kv) / scales[kv]
                kk = pool[layer, 0, page, :, off] * scales[0]
                vv = pool[layer, 1, page, :, off] * scales[1]
                out.append(_attend(cfg, layer, q[b:b + 1], pos[b:b + 1], kk, vv))
            x = _finish_layer(cfg, lw, x, torch.cat(out))
        return {"logits": _logits(cfg, w, x), "pool": pool.reshape(-1)}

    x = w["embed"][torch.as_tensor(tokens, device=dev).long()].double()
    if visual is not None:
        first = 64 if 64 + len(visual) <= lens[0] else 0
        x[first:first + len(visual)] = visual.double()
    pos = torch.cat([torch.arange(n, device=dev) for n in lens])
    last = torch.as_tensor([int(starts[b + 1]) - 1 for b in range(len(lens))], device=dev)
    for layer, lw in enumerate(w["layers"]):
        kept = layer < case["l_keep"]
        if kept:
            q, k, v = _qkv(cfg, lw, layer, x, pos)
        else:
            # a pruned layer: the body leaves its keys and values only, the last tokens run it in full
            if layer == case["l_keep"]:
                xl = x[last]
            _, k, v = _qkv(cfg, lw, layer, x, pos)
            ql, kl, vl = _qkv(cfg, lw, layer, xl, pos[last])
            k[last], v[last] = kl, vl
        out = []
        for b, n in enumerate(lens):
            r = slice(int(starts[b]), int(starts[b + 1]))
            page, off = places(b, n)
            pool[layer, 0, page, :, off] = k[r]
            pool[layer, 1, page, :, off] = v[r]
            out.append(_attend(cfg, layer, q[r] if kept else ql[b:b + 1], pos[r] if kept else pos[last][b:b + 1], k[r], v[r]))
        if kept:
            x = _finish_layer(cfg, lw, x, torch.cat(out))
        else:
            xl = _finish_layer(cfg, lw, xl, torch.cat(out))
    if case["l_keep"] >= cfg["n_layers"]:
        xl = x[last]
    return {"logits": _logits(cfg, w, xl), "pool": pool.reshape(-1)}
