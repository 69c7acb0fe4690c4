"""The work that a user of this library has it do, as cases that can be timed and checked.

Every case is one request through the public calls of the binding: a prompt, and what follows it -- nothing but the first
token's logits ("prompt"), greedy decoding with the full model ("vanilla"), self-speculative cycles of draft, verification,
acceptance and per-layer confidence ("ssd"), or cycles followed by the confidence of the whole context window ("window").
A case has the widths of one of the repository's workloads and, except for the two whole models, its first few layers
only: rounding travels through the layers, so the tolerances of shallow stacks are tight.

Weights are drawn from the seed: N(0, 0.02) matrices, the projections back into the residual stream scaled by
1/sqrt(2 depth), embeddings N(0, 1) and norm gains around 1.  The LM head answers an embedding with one successor token
(a seeded permutation of the vocabulary) well above its noise, as a trained model answers most positions with confidence:
the greedy tokens do not hang on the last bits of the logits, drafts are accepted, and soft-max and entropy see a peak.
"""
import math

import numpy as np
import torch

import paper_2604_14612_amd as ssd

# widths of the repository's workloads: d_model, heads, KV heads, FFN, vocabulary, rotary base, full depth
MODELS = {
    "tiny": (256, 4, 4, 688, 1024, 1e4, 4),
    "small": (1024, 16, 16, 2816, 32000, 1e4, 24),
    "llama7b": (4096, 32, 32, 11008, 32000, 1e4, 32),
    "llama3_8b": (4096, 32, 8, 14336, 128256, 5e5, 32),
    "llama13b": (5120, 40, 40, 13824, 32000, 1e4, 40),
    "llama70b": (8192, 64, 8, 28672, 32000, 1e4, 80),
}
DTYPES = {"fp32": torch.float32, "bf16": torch.bfloat16, "fp16": torch.float16}
RMS_EPS, CONF_EPS = 1e-5, 1e-10
PEAK = 16.0     # height of the successor's row in the LM head, in units of the row noise


class Shape:
    """The attributes a Context asks of a model shape."""

    def __init__(self, case):
        d, h, hkv, f, v, base, _ = MODELS[case["model"]]
        self.n_layers, self.d_model, self.n_heads, self.n_kv_heads, self.d_ffn, self.vocab = case["layers"], d, h, hkv, f, v
        self.head_dim, self.d_kv, self.dtype, self.rms_eps, self.rope_base = d // h, d // h * hkv, case["dtype"], RMS_EPS, base


# ---- the cases -----------------------------------------------------------------------------------------------------

def listed():
    c = lambda name, op, model, layers, dtype, kv, prompt, steps, k: dict(  # noqa: E731
        name=name, op=op, model=model, layers=layers, dtype=dtype, kv=kv, prompt=prompt, steps=steps, k=k)
    return [
        # the smallest model, fp32 throughout: launches and latency only
        c("tiny-fp32-ssd", "ssd", "tiny", 4, "fp32", "fp32", 32, 7, 4),
        # a whole small model answering a request token by token
        c("small-vanilla", "vanilla", "small", 24, "bf16", "fp32", 256, 48, 0),
        # the same widths, shallow, speculating
        c("small-ssd-k4", "ssd", "small", 8, "bf16", "fp32", 200, 12, 4),
        # the headline widths: the prompt pass, and greedy decoding behind it
        c("7b-prompt-512", "prompt", "llama7b", 4, "bf16", "fp32", 512, 0, 0),
        c("7b-vanilla", "vanilla", "llama7b", 6, "bf16", "fp32", 100, 40, 0),
        # the headline itself: the whole 7B model, a 512-token prompt, draft length 4
        c("7b-whole-ssd-k4", "ssd", "llama7b", 32, "bf16", "fp32", 512, 8, 4),
        # half-precision weights and cache, the longest draft of the sweep, an odd prompt
        c("7b-f16-ssd-k8", "ssd", "llama7b", 4, "fp16", "fp16", 77, 8, 8),
        # the search's confidence over the context window, taps of every committed position
        c("7b-window", "window", "llama7b", 6, "bf16", "fp32", 60, 12, 7),
        # grouped heads and a large vocabulary: a chat turn
        c("8b-vanilla", "vanilla", "llama3_8b", 3, "bf16", "bf16", 45, 32, 0),
        # a long document, then an answer over its cache
        c("8b-long", "vanilla", "llama3_8b", 2, "bf16", "bf16", 4001, 32, 0),
        # a ragged prompt at the 13B widths
        c("13b-prompt-1000", "prompt", "llama13b", 3, "bf16", "fp32", 1000, 0, 0),
        # the largest widths, speculating behind a medium prompt
        c("70b-ssd-k4", "ssd", "llama70b", 3, "bf16", "fp32", 300, 8, 4),
    ]


def _cost(case):
    """Rough seconds of a pass (for draw: no dearer than the dearest listed case)."""
    w = work(case)
    per_step = case["layers"] * 5 * (case["k"] + 1) + 30
    return w["flops"] / 300e12 + w["bytes"] / 4e12 + case["steps"] * per_step * 4e-6


def draw(rng):
    limit = max(_cost(c) for c in listed())
    while True:
        model = rng.choice(sorted(MODELS))
        op = rng.choice(("prompt", "vanilla", "vanilla", "ssd", "ssd", "ssd", "window"))
        dtype = "fp32" if model == "tiny" else rng.choice(("bf16", "bf16", "fp16"))
        kv = "fp32" if dtype == "fp32" else rng.choice(("fp32", "fp32", dtype))
        case = {
            "op": op, "model": model, "layers": rng.randint(1, 4) if model != "small" else rng.randint(4, 24), "dtype": dtype, "kv": kv,
            "prompt": int(round(math.exp(rng.uniform(math.log(2), math.log(4096))))),
            "steps": 0 if op == "prompt" else rng.randint(4, 32) if op == "vanilla" else rng.randint(2, 12),
            "k": 0 if op in ("prompt", "vanilla") else rng.choice((1, 2, 3, 4, 4, 5, 6, 8, 8, 11, 15)),
        }
        if _cost(case) <= limit:
            return case


# ---- weights and inputs ----------------------------------------------------------------------------------------------

def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _randn(shape, seed, layer, tid, dtype):
    g = torch.Generator(device=_device())
    g.manual_seed((seed * 1000003 + (layer + 1) * 131 + tid) & 0x7FFFFFFF)
    return torch.randn(shape, generator=g, device=_device(), dtype=torch.float32).to(dtype)


def _layer(case, seed, l):
    d, h, hkv, f, _, _, depth = MODELS[case["model"]]
    dt, dkv, res = DTYPES[case["dtype"]], d // h * hkv, 0.02 / math.sqrt(2.0 * depth)
    m = lambda n, k, std, tid: _randn((n, k), seed, l, tid, torch.float32).mul_(std).to(dt)  # noqa: E731
    gain = lambda tid: _randn((d,), seed, l, tid, torch.float32).mul_(0.1).add_(1.0)  # noqa: E731
    return {"attn_norm": gain(0), "wq": m(d, d, 0.02, 1), "wk": m(dkv, d, 0.02, 2), "wv": m(dkv, d, 0.02, 3), "wo": m(d, d, res, 4),
            "mlp_norm": gain(5), "wg": m(f, d, 0.02, 6), "wu": m(f, d, 0.02, 7), "wd": m(d, f, res, 8)}


def _ends(case, seed):
    """Embedding, LM head, final gain, and the successor of every token."""
    d, _, _, _, v, _, _ = MODELS[case["model"]]
    dt = DTYPES[case["dtype"]]
    embed = _randn((v, d), seed, -1, 20, dt)
    succ = torch.from_numpy(np.random.RandomState(seed & 0x7FFFFFFF).permutation(v))
    head = _randn((v, d), seed, -1, 21, torch.float32).mul_(0.02)
    where = succ.to(head.device)
    for a in range(0, v, 16384):      # in pieces: no second fp32 copy of a large vocabulary
        e = embed[a:a + 16384].float()
        head[where[a:a + 16384]] += e * (0.02 * PEAK / e.norm(dim=1, keepdim=True))
    final = _randn((d,), seed, -1, 22, torch.float32).mul_(0.1).add_(1.0)
    return embed, head.to(dt), final, succ.numpy()


def _prompt(case, seed):
    v = MODELS[case["model"]][4]
    return np.random.RandomState((seed + 17) & 0x7FFFFFFF).randint(0, v, case["prompt"]).astype(np.int32)


def _mask(case):
    """Uniform skipping: every second layer, the first one kept."""
    return np.array([l % 2 for l in range(case["layers"])], np.uint8)


def _new_tokens(case):
    return 1 + case["steps"] * (case["k"] + 1)


def prepare(case, seed):
    w = {}
    for l in range(case["layers"]):
        for name, t in _layer(case, seed, l).items():
            w.setdefault(name, []).append(t)
    w["embed"], w["lm_head"], w["final_norm"], _ = _ends(case, seed)
    w = ssd.pack_weights(w)
    window = {"conf_window": 100} if case["op"] == "window" else {}
    ctx = ssd.Context(Shape(case), w, case["prompt"] + _new_tokens(case) + 16, max(case["k"], 1), kv_dtype=case["kv"], **window)
    return {"case": case, "ctx": ctx, "prompt": _prompt(case, seed).tolist(), "mask": _mask(case)}


def run(state):
    case, ctx = state["case"], state["ctx"]
    ctx.ssd_reset()
    if case["op"] == "vanilla":
        tokens = ssd.generate_vanilla(ctx, state["prompt"], case["steps"] + 1)
        return {"tokens": np.array(tokens, np.int32), "logits": ctx.ssd_copy_logits(0, 1)}
    tokens = [ctx.ssd_prefill(state["prompt"])]
    if case["op"] == "prompt":
        return {"tokens": np.array(tokens, np.int32), "logits": ctx.ssd_copy_logits(0, 1)}
    k, out = case["k"], {}
    for i in range(case["steps"]):
        draft = ctx.ssd_draft_step(state["mask"], k)
        target = ctx.ssd_verify(draft)
        a, nxt = ctx.ssd_accept(draft, target)
        tokens += draft[:a] + [nxt]
        if i + 1 == case["steps"]:
            out["logits"] = ctx.ssd_copy_logits(0, k + 1)
        if case["op"] == "ssd":
            out["confidence"] = ctx.ssd_layer_confidence(0, 1)[0]
    if case["op"] == "window":
        out["confidence"] = ctx.ssd_window_confidence()
    out["tokens"] = np.array(tokens, np.int32)
    return out


# ---- what a pass cannot do without -----------------------------------------------------------------------------------

def work(case):
    d, h, hkv, f, v, _, _ = MODELS[case["model"]]
    L, n, k, steps = case["layers"], case["prompt"], case["k"], case["steps"]
    B, Bkv = (4 if case["dtype"] == "fp32" else 2), (4 if case["kv"] == "fp32" else 2)
    dkv = d // h * hkv
    par = 2 * d * d + 2 * d * dkv + 3 * d * f

    def rows(layers, r, p):
        """r rows behind p cached positions through `layers` layers: weights once, cache read and written, attention."""
        att = layers * 4 * d * (r * p + r * (r + 1) / 2)
        return layers * (par * B + 2 * (p + r) * dkv * Bkv) + r * d * B, layers * 2 * par * r + att

    bytes_, flops = rows(L, n, 0)
    bytes_, flops = bytes_ + v * d * B + 4 * v, flops + 2 * v * d
    pos = n
    executed = L - int(_mask(case).sum())
    for _ in range(steps):
        if case["op"] == "vanilla":
            b, fl = rows(L, 1, pos)
            bytes_, flops, pos = bytes_ + b + v * d * B, flops + fl + 2 * v * d, pos + 1
            continue
        for i in range(k):
            b, fl = rows(executed, 1, pos + i)
            bytes_, flops = bytes_ + b + v * d * B, flops + fl + 2 * v * d
        b, fl = rows(L, k + 1, pos)
        bytes_, flops = bytes_ + b + v * d * B + 2 * L * d * 4 * (k + 1), flops + fl + 2 * v * d * (k + 1)
        if case["op"] == "ssd":
            bytes_, flops = bytes_ + v * d * B + 2 * L * d * 4, flops + 2 * v * d * 2 * L
        pos += k + 1
    if case["op"] == "window":
        p = min(100, 1 + steps * (k + 1))
        bytes_, flops = bytes_ + v * d * B + p * 2 * L * d * 4, flops + 2 * v * d * 2 * L * p
    return {"bytes": float(bytes_), "flops": float(flops)}


def tolerance(case):
    # measured against exact(): 1.3e-6 (fp32), 7e-6 (16-bit weights, fp32 cache), 7e-5 (fp16 cache), 3e-4 (bf16 cache)
    return {"rel": {"fp32": 1e-5 if case["dtype"] == "fp32" else 4e-5, "fp16": 3e-4, "bf16": 2e-3}[case["kv"]]}


# ---- the same in 64 bits -----------------------------------------------------------------------------------------------

def exact(case, seed):
    d, h, hkv, f, v, base, _ = MODELS[case["model"]]
    hd, G = d // h, h // hkv
    dev = _device()
    embed, head, final, succ = _ends(case, seed)
    # the greedy continuation is the chain of successors; checked against the 64-bit logits below
    seq = _prompt(case, seed).tolist()
    n, total = len(seq), len(seq) + (_new_tokens(case) if case["op"] != "vanilla" else case["steps"] + 1)
    while len(seq) < total:
        seq.append(int(succ[seq[-1]]))
    T = total - 1                                     # the last token is never fed
    x = embed[torch.tensor(seq[:T], device=dev)].double()
    ang = torch.arange(T, dtype=torch.float64, device=dev)[:, None] * torch.pow(
        torch.tensor(float(base), dtype=torch.float64, device=dev), -torch.arange(0, hd, 2, dtype=torch.float64, device=dev) / hd)[None]
    cos, sin = ang.cos()[:, None], ang.sin()[:, None]

    def norm(t, g):
        return t * torch.rsqrt(t.square().mean(-1, keepdim=True) + RMS_EPS) * g.double()

    def rotate(t):
        a, b = t[..., :hd // 2], t[..., hd // 2:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)

    if case["op"] == "window":                        # positions fed with committed tokens: the last prompt one, then every verify row
        conf_rows = list(range(max(n - 1, T - 100), T))
    elif case["op"] == "ssd":                         # the first row of the last verification
        conf_rows = [T - case["k"] - 1]
    else:
        conf_rows = []
    taps = []
    for l in range(case["layers"]):
        w = _layer(case, seed, l)
        y = norm(x, w["attn_norm"])
        q = rotate((y @ w["wq"].double().t()).view(T, h, hd)).transpose(0, 1).contiguous()
        kk = rotate((y @ w["wk"].double().t()).view(T, hkv, hd)).transpose(0, 1).contiguous()
        vv = (y @ w["wv"].double().t()).view(T, hkv, hd).transpose(0, 1).contiguous()
        out = torch.empty(h, T, hd, dtype=torch.float64, device=dev)
        for i in range(h):
            for a in range(0, T, 1024):
                e = min(T, a + 1024)
                s = q[i, a:e] @ kk[i // G, :e].t() / math.sqrt(hd)
                s.masked_fill_(torch.arange(e, device=dev)[None] > torch.arange(a, e, device=dev)[:, None], -math.inf)
                out[i, a:e] = torch.softmax(s, -1) @ vv[i // G, :e]
        x = x + out.transpose(0, 1).reshape(T, d) @ w["wo"].double().t()
        taps.append(x[conf_rows])
        y = norm(x, w["mlp_norm"])
        x = x + (torch.nn.functional.silu(y @ w["wg"].double().t()) * (y @ w["wu"].double().t())) @ w["wd"].double().t()
        taps.append(x[conf_rows])
    # logits of the generated positions
    z = norm(x[n - 1:], final) @ head.double().t()
    if z.argmax(-1).tolist() != seq[n:]:
        return None
    rows = 1 if case["op"] in ("prompt", "vanilla") else case["k"] + 1
    got = {"tokens": np.array(seq[n:], np.int32), "logits": z[-rows:].cpu().numpy()}
    if conf_rows:
        per_tap = []
        for t in taps:
            p = torch.softmax(norm(t, final) @ head.double().t(), -1)
            per_tap.append((1.0 + (p * torch.log(p + CONF_EPS)).sum(-1) / math.log(v)).mean())
        conf = torch.stack(per_tap).view(case["layers"], 2).mean(-1)
        got["confidence"] = conf.cpu().numpy()
    return got
