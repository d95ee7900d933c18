"""The work a user of this library has it do, as cases that can be timed and compared.

Each case is one pass through the public entry points: a model loaded into a
GpuModel, a KV cache with a context in it, and one call that decodes
(``GpuModel.step``, ``GpuModel.greedy`` or ``kl_decode_step_noalloc``).  The
library runs decode only: prefill and training are no part of it.  The model
shapes are those of ``synth.workloads``; where a whole model would only repeat
the same layer, a case runs a few of its layers with its whole classifier, so
that the case stays near a layer's own cost and the inputs are quick to make.
Weights, caches and tokens are seeded normal and uniform values of the
distributions the library's own workloads use.
"""
from __future__ import annotations

import math

import torch

from paper_2410_23668_amd import binding as kb
from paper_2410_23668_amd.device import GpuModel, KvCache, stream_handle
from synth.workloads import LLAMA3B, LLAMA70B, LLAMA8B, MIXTRAL, QWEN72B, TINY

_FIELDS = dict(layers="n_layers", hidden="hidden", heads="n_heads", kv_heads="n_kv_heads",
               head_dim="head_dim", ffn="ffn_dim", vocab="vocab", theta="rope_theta",
               eps="rms_eps")


def _case(model: dict, batch: int, context: int, layers: int = 0, ragged: bool = False,
          call: str = "step", steps: int = 1, **named) -> dict:
    c = {k: model[v] for k, v in _FIELDS.items()}
    c["layers"] = layers or model["n_layers"]
    c.update(tied=bool(model.get("tie_embeddings", False)), bias=bool(model.get("qkv_bias", False)),
             experts=model.get("n_experts", 0), top_k=model.get("top_k", 0), batch=batch,
             context=context, ragged=ragged, call=call, steps=steps, **named)
    return c


def listed() -> list:
    return [
        # the smallest call: a toy model, where the latency of a step is all there is
        _case(TINY, 1, 128, name="tiny b1"),
        # one user of an 8B chat model: the whole model (the library's headline)
        _case(LLAMA8B, 1, 4096, name="8b b1"),
        # a greedy token loop of a small model, tokens fed back on the device
        _case(LLAMA3B, 1, 2048, call="greedy", steps=8, name="3b b1 greedy"),
        # a long document: the cache is a large share of what is read
        _case(LLAMA8B, 1, 32768, layers=8, name="8b b1 long"),
        # a few users with prompts of different lengths
        _case(LLAMA8B, 3, 1500, layers=8, ragged=True, name="8b b3 ragged"),
        _case(LLAMA8B, 4, 4096, layers=8, name="8b b4"),
        # an odd number of requests in a lightly loaded server
        _case(LLAMA8B, 7, 2999, layers=8, ragged=True, name="8b b7 ragged"),
        # a busy server
        _case(LLAMA8B, 16, 8192, layers=8, name="8b b16"),
        _case(LLAMA8B, 32, 4096, layers=8, ragged=True, name="8b b32 ragged"),
        # a large model: one user, and a full batch
        _case(LLAMA70B, 1, 4096, layers=4, name="70b b1"),
        _case(LLAMA70B, 32, 4096, layers=4, name="70b b32"),
        # a mixture of experts
        _case(MIXTRAL, 1, 4096, layers=4, name="mixtral b1"),
    ]


def _log(rng, lo: int, hi: int) -> int:
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _generic(rng) -> dict:
    """A model of no name: any supported head dimension and grouping, odd widths."""
    d = rng.choice((64, 128))
    kv = rng.randint(1, 8)
    group = rng.choice((1, 2, 4, 8) if d == 64 else (1, 2, 3, 4, 8))
    return dict(n_layers=1, hidden=8 * _log(rng, 16, 512), n_heads=kv * group, n_kv_heads=kv,
                head_dim=d, ffn_dim=8 * _log(rng, 32, 1536), vocab=_log(rng, 500, 60000),
                rope_theta=10000.0, rms_eps=1e-5, qkv_bias=rng.random() < 0.3,
                tie_embeddings=rng.random() < 0.3)


def draw(rng) -> dict:
    while True:
        model = rng.choice((LLAMA8B, LLAMA8B, LLAMA3B, LLAMA70B, QWEN72B, MIXTRAL, None, None))
        moe = model is MIXTRAL
        big = model is LLAMA70B or model is QWEN72B
        batch = _log(rng, 1, 7 if moe else 40)
        layers = rng.randint(1, 3 if big or moe else 8)
        if model is None:
            model = _generic(rng)
        context = _log(rng, 24, 40000)
        call = rng.choice(("step", "step", "step", "step", "greedy", "noalloc"))
        if call == "noalloc" and batch > 4:   # (the static scratch is for small steps)
            call = "step"
        steps = rng.randint(2, 6) if call == "greedy" else 1
        c = _case(model, batch, context, layers=layers, ragged=rng.random() < 0.6, call=call,
                  steps=steps)
        if work(c)["bytes"] <= 9e9:
            return c


# ---------------------------------------------------------------- inputs

def _model(c: dict) -> dict:
    m = {v: c[k] for k, v in _FIELDS.items()}
    m["qkv_bias"] = c["bias"]
    if c["experts"]:
        m.update(n_experts=c["experts"], top_k=c["top_k"])
    return m


def _capacity(c: dict) -> int:
    return (c["context"] + c["steps"] + 63) // 64 * 64


def _contexts(c: dict) -> list:
    """Cached positions of each sequence; ragged: spread from the whole context to half of it."""
    n, b = c["context"], c["batch"]
    return [n - (n // 2) * i // b if c["ragged"] else n for i in range(b)]


def _normal(seed: int, stream: int, shapes: dict) -> dict:
    g = torch.Generator(device="cuda").manual_seed(1_000_003 * seed + stream)
    out = {}
    for name, (shape, std, mean) in shapes.items():
        t = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
        out[name] = t.normal_(mean, std, generator=g)
    return out


def _layer(c: dict, seed: int, l: int) -> dict:
    H, F, E = c["hidden"], c["ffn"], c["experts"]
    Q, KV = c["heads"] * c["head_dim"], c["kv_heads"] * c["head_dim"]
    ex = (E,) if E else ()
    s = dict(attn_norm=((H,), 0.01, 1.0), wq=((Q, H), 0.02, 0.0), wk=((KV, H), 0.02, 0.0),
             wv=((KV, H), 0.02, 0.0), wo=((H, Q), 0.02, 0.0), ffn_norm=((H,), 0.01, 1.0),
             w_gate=(ex + (F, H), 0.02, 0.0), w_up=(ex + (F, H), 0.02, 0.0),
             w_down=(ex + (H, F), 0.02, 0.0))
    if c["bias"]:
        s.update(bq=((Q,), 0.5, 0.0), bk=((KV,), 0.5, 0.0), bv=((KV,), 0.5, 0.0))
    if E:
        s["w_router"] = ((E, H), 0.02, 0.0)
    return _normal(seed, 1 + l, s)


def _globals(c: dict, seed: int) -> dict:
    V, H = c["vocab"], c["hidden"]
    s = dict(embed=((V, H), 0.02, 0.0), final_norm=((H,), 0.01, 1.0))
    if not c["tied"]:
        s["lm_head"] = ((V, H), 0.02, 0.0)
    g = _normal(seed, 0, s)
    g.setdefault("lm_head", g["embed"])
    return g


def _cache(c: dict, seed: int, l: int) -> dict:
    shape = (c["batch"], c["kv_heads"], _capacity(c), c["head_dim"])
    return _normal(seed, 100_000 + l, dict(k=(shape, 1.0, 0.0), v=(shape, 1.0, 0.0)))


def _tokens(c: dict, seed: int) -> torch.Tensor:
    g = torch.Generator().manual_seed(1_000_003 * seed + 200_000)
    return torch.randint(0, c["vocab"], (c["batch"],), generator=g, dtype=torch.int32).cuda()


def prepare(case: dict, seed: int) -> dict:
    c, m = case, _model(case)
    B = c["batch"]
    model = GpuModel.from_layers(m, lambda l: _layer(c, seed, l), lambda: _globals(c, seed),
                                 max_batch=B, max_seq=_capacity(c))
    kv = KvCache(m, B, _capacity(c))
    for l in range(c["layers"]):
        new = _cache(c, seed, l)
        kv.k[l].copy_(new["k"].view(torch.int16))
        kv.v[l].copy_(new["v"].view(torch.int16))
    s = dict(case=c, model=model, kv=kv, tokens=_tokens(c, seed),
             positions=torch.tensor(_contexts(c), dtype=torch.int32, device="cuda"),
             logits=torch.empty(B, c["vocab"], dtype=torch.float32, device="cuda"))
    if c["call"] == "greedy":
        s["out"] = torch.empty(c["steps"], B, dtype=torch.int32, device="cuda")
    else:
        s["hidden"] = torch.empty(B, c["hidden"], dtype=torch.float32, device="cuda")
    return s


def run(state: dict) -> dict:
    s, model, kv = state, state["model"], state["kv"]
    out = dict(logits=s["logits"], k=kv.k.view(torch.bfloat16), v=kv.v.view(torch.bfloat16))
    if s["case"]["call"] == "greedy":
        model.greedy(s["tokens"], s["positions"], kv, s["case"]["steps"], s["out"], s["logits"],
                     kb.KL_MODE_LOOPED)
        out["tokens"] = s["out"]
        return out
    out["hidden"] = s["hidden"]
    if s["case"]["call"] == "step":
        model.step(s["tokens"], s["positions"], kv, s["logits"], s["hidden"], kb.KL_MODE_LOOPED)
    else:
        kb.kl_decode_step_noalloc(model.state, s["tokens"].data_ptr(), s["positions"].data_ptr(),
                                  s["case"]["batch"], kv.k.data_ptr(), kv.v.data_ptr(), kv.batch,
                                  kv.capacity, s["logits"].data_ptr(), s["hidden"].data_ptr(),
                                  stream_handle(), kb.KL_MODE_LOOPED)
    return out


# ---------------------------------------------------------------- what a pass has to do

def work(case: dict) -> dict:
    """Every weight once per step (with experts: those the batch is expected to
    choose), the cached keys and values up to each position, one embedding row
    per sequence, the new cache slots, the logits and the hidden state."""
    c, B, H, d = case, case["batch"], case["hidden"], case["head_dim"]
    Q, KV, F, V = c["heads"] * d, c["kv_heads"] * d, c["ffn"], c["vocab"]
    attn = H * (2 * Q + 2 * KV) + (Q + 2 * KV if c["bias"] else 0)
    E, k = c["experts"], c["top_k"]
    used = E * (1.0 - (1.0 - k / E) ** B) if E else 1.0
    mlp, router = 3 * H * F, E * H
    per_token = attn + mlp * (k if E else 1) + router
    nbytes = flops = 0.0
    for s in range(c["steps"]):
        pos = [n + s for n in _contexts(c)]
        nbytes += 2 * (c["layers"] * (attn + mlp * used + router + 2 * H) + H + V * H)
        nbytes += 2 * B * H + c["layers"] * sum(4 * KV * (p + 1) for p in pos)
        nbytes += 4 * B * (V + (H if c["call"] != "greedy" else 0))
        flops += 2 * B * (c["layers"] * per_token + V * H)
        flops += c["layers"] * sum(4 * Q * (p + 1) for p in pos)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case: dict) -> dict:
    # rel: about four times the largest error measured against 64 bits over
    # listed and drawn cases: fp32 sums up to batch 4 (3e-6 through 32 layers,
    # 3e-5 in a token loop), two-term bf16 products above (2e-5; 2e-4 at
    # contexts of a few dozen positions, where the last bit of a new bf16
    # cache entry shows).  max: one rounding step of such an entry.
    # differ: tokens of a greedy loop, for ties.
    small = case["batch"] <= 4 and case["call"] != "greedy"
    return {"rel": 2e-4 if small else 8e-4, "max": 0.01, "differ": 0.01}


# ---------------------------------------------------------------- the same in 64 bits

def _norm64(x, gain, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * gain.double()


def _mlp64(c, w, h):
    def one(gate, up, down, y):
        g = y @ gate.double().t()
        return (g / (1 + torch.exp(-g)) * (y @ up.double().t())) @ down.double().t()
    if not c["experts"]:
        return one(w["w_gate"], w["w_up"], w["w_down"], h)
    out = torch.zeros_like(h)
    logit = h @ w["w_router"].double().t()
    for b in range(h.shape[0]):
        top = torch.sort(logit[b], descending=True, stable=True).indices[:c["top_k"]].tolist()
        share = torch.softmax(logit[b][top], 0)
        for e, p in zip(top, share):
            out[b] += p * one(w["w_gate"][e], w["w_up"][e], w["w_down"][e], h[b:b + 1])[0]
    return out


def _step64(c, layer, globs, caches, tokens, positions):
    """One decode step in 64 bits; the new keys and values are rounded to the
    cache's bf16 and put in its slots."""
    d, nq, nkv, B = c["head_dim"], c["heads"], c["kv_heads"], c["batch"]
    x = globs["embed"][tokens.long()].double()
    freq = c["theta"] ** (-2.0 * torch.arange(d // 2, dtype=torch.float64, device="cuda") / d)
    phi = torch.tensor(positions, dtype=torch.float64, device="cuda")[:, None, None] * freq
    cos, sin = torch.cos(phi), torch.sin(phi)

    def rope(t):
        a, b = t[..., :d // 2], t[..., d // 2:]
        return torch.cat((a * cos - b * sin, a * sin + b * cos), -1)

    for l in range(c["layers"]):
        w, kv = layer(l), caches(l)
        h = _norm64(x, w["attn_norm"], c["eps"])
        q, k, v = (h @ w[n].double().t() + (w[b].double() if c["bias"] else 0.0)
                   for n, b in (("wq", "bq"), ("wk", "bk"), ("wv", "bv")))
        q, k = rope(q.view(B, nq, d)), rope(k.view(B, nkv, d))
        v = v.view(B, nkv, d)
        o = torch.empty(B, nkv, nq // nkv, d, dtype=torch.float64, device="cuda")
        for b, p in enumerate(positions):
            kv["k"][b, :, p] = k[b].to(torch.bfloat16)
            kv["v"][b, :, p] = v[b].to(torch.bfloat16)
            K, W = (kv[n][b, :, :p + 1].double() for n in ("k", "v"))
            s = torch.matmul(q[b].view(nkv, nq // nkv, d), K.transpose(1, 2).contiguous())
            o[b] = torch.matmul(torch.softmax(s / math.sqrt(d), -1), W)
        x = x + o.view(B, nq * d) @ w["wo"].double().t()
        x = x + _mlp64(c, w, _norm64(x, w["ffn_norm"], c["eps"]))
    h = _norm64(x, globs["final_norm"], c["eps"])
    logits = torch.empty(B, c["vocab"], dtype=torch.float64, device="cuda")
    for r in range(0, c["vocab"], 16384):
        logits[:, r:r + 16384] = h @ globs["lm_head"][r:r + 16384].double().t()
    return logits, x


def exact(case: dict, seed: int) -> dict:
    """run() in 64 bits, by plain torch.  The caches are left out: their new
    slots are rounded to bf16, where a last bit of the sum may go either way."""
    c, globs, tokens = case, _globals(case, seed), _tokens(case, seed)
    keep = c["steps"] > 1   # (a token loop comes back to its layers)
    layers = [_layer(c, seed, l) for l in range(c["layers"])] if keep else None
    caches = [_cache(c, seed, l) for l in range(c["layers"])] if keep else None
    out, picked = dict(k=None, v=None), []
    for s in range(c["steps"]):
        logits, x = _step64(c, layers.__getitem__ if keep else lambda l: _layer(c, seed, l), globs,
                            caches.__getitem__ if keep else lambda l: _cache(c, seed, l), tokens,
                            [n + s for n in _contexts(c)])
        tokens = logits.argmax(-1)
        picked.append(tokens.to(torch.int32))
    out["logits"] = logits
    if c["call"] == "greedy":
        out["tokens"] = torch.stack(picked)
    else:
        out["hidden"] = x
    return out
