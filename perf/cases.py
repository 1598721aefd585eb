"""The calls whose speed this repository is measured by, and plain float64 references of them.

Every case is a call of the decoder forward (`Model.forward`, sd_forward of the
C ABI) over a KV cache the caller owns, on a model of one of the LLaMA-2 shapes
this repository decodes (7B, 13B, 70B with grouped-query heads; bfloat16) or on
the tiny float32 model.  A forward is what every decoding step runs: one row is
a draft step (with a skip mask) or an autoregressive step, 2 to 16 rows a
verification, more rows a prompt prefill or the scoring of a text.  Most cases
run a few layers of the shape and the head, so that the layers' own rounding
shows; one is the whole 13B model up to its first token.

A case is {"name", "model", "layers", "rows", "ctx", "cap", "skip", "fp8",
"first"}: `rows` tokens after `ctx` cached positions of a cache of `cap`
positions, bypassing the sublayers listed in `skip` (2l: attention of layer l,
2l + 1: its MLP).  "fp8": the draft's weights are quantized (a one-row draft
step).  "first": the rows are prefilled without logits, as a generate call
does, and one more row gives the logits of the first new token.
"""

import math
import types

import numpy as np
import torch

from paper_2309_08168_amd import binding

SHAPES = {
    # layers of the whole model, d_model, heads, kv heads, head_dim, ffn, vocabulary, type
    "tiny": (4, 256, 4, 4, 64, 688, 1024, "f32"),
    "7b": (32, 4096, 32, 32, 128, 11008, 32000, "bf16"),
    "13b": (40, 5120, 40, 40, 128, 13824, 32000, "bf16"),
    "70b": (80, 8192, 64, 8, 128, 28672, 32000, "bf16"),
}
EPS, ROPE_BASE = 1e-6, 10000.0


def _case(name, model, layers, rows, ctx, cap, skip="", fp8=False, first=False):
    c = {"model": model, "layers": layers, "rows": rows, "ctx": ctx, "cap": cap, "skip": skip, "fp8": fp8,
         "first": first}
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest call: a full stage's verification (4 drafts) of the tiny float32 model; latency only.
        _case("tiny verify 5 rows", "tiny", 4, 5, 30, 64),
        # A draft step: one row, a quarter of the sublayers skipped, in the middle of a 1024 + 512 token decode.
        _case("13b draft 1 row", "13b", 4, 1, 1200, 1550, "2,5"),
        # The same draft step on FP8 copies of the draft's weights.
        _case("13b draft fp8", "13b", 4, 1, 1200, 1550, "2,5", fp8=True),
        # The verification of one draft, early in a decode, in a cache as large as the model's context.
        _case("7b verify 2 rows", "7b", 4, 2, 600, 4096),
        # The verification of a short stage (3 drafts).
        _case("13b verify 4 rows", "13b", 4, 4, 1200, 1550),
        # The verification of a full stage, K_max 12.
        _case("13b verify 13 rows", "13b", 4, 13, 1500, 1550),
        # The verification of a full stage with grouped-query heads, K_max 8.
        _case("70b verify 9 rows", "70b", 2, 9, 580, 650),
        # An autoregressive step at the end of a long document: as many KV bytes as weights.
        _case("13b step 1 row, 30k keys", "13b", 4, 1, 30000, 32768),
        # A short question: the prompt of a chat turn.
        _case("13b prompt 33 rows", "13b", 4, 33, 0, 256),
        # The 7B workload's prompt.
        _case("7b prompt 511 rows", "7b", 4, 511, 0, 768),
        # One chunk of a long document's prefill, an attention-heavy one.
        _case("13b prompt 1000 at 8k", "13b", 4, 1000, 8000, 9216),
        # Time to the first token of the 13B workload: the whole model over its 1024-token prompt.
        _case("13b first token, 1024", "13b", 40, 1023, 0, 1550, first=True),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["tiny", "step", "verify", "verify", "prompt", "prompt", "prompt"])
    model = "tiny" if kind == "tiny" else rng.choice(["7b", "13b", "13b", "70b"])
    layers = rng.randint(1, 2 if model == "70b" else 4)
    rows = {"tiny": log_int(1, 40), "step": 1, "verify": rng.randint(2, 16), "prompt": log_int(17, 1400)}[kind]
    ctx = 0 if kind == "prompt" and rng.random() < 0.5 else log_int(20, 400 if kind == "tiny" else 20000)
    cap = ctx + rows + log_int(8, 4000)
    skip = [i for i in range(2 * layers) if rng.random() < (0.25 if rng.random() < 0.5 else 0.0)]
    fp8 = kind == "step" and rng.random() < 0.3
    return _case(None, model, layers, rows, ctx, cap, ",".join(map(str, skip)), fp8)


# ----------------------------------------------------------------------------
# inputs


def _config(case):
    L, d, H, KVH, dh, F, V, dtype = SHAPES[case["model"]]
    return types.SimpleNamespace(n_layers=case["layers"], d_model=d, n_heads=H, n_kv_heads=KVH, head_dim=dh, ffn_dim=F,
                                 vocab=V, dtype=dtype, rms_eps=EPS, rope_base=ROPE_BASE)


def _skip(case):
    z = np.zeros(2 * case["layers"], np.uint8)
    for i in case["skip"].split(","):
        if i:
            z[int(i)] = 1
    return z


def _masked(case):
    return bool(case["skip"]) or case["fp8"]


def _inputs(case, seed):
    """(weights by name, cache [L][2][KVH][cap][dh], token ids), from the seed alone: linear weights and the embedding
    N(0, 0.02^2), the output projections scaled down by the depth, gains around 1, cached keys and values N(0, 1)."""
    c = _config(case)
    dt = torch.bfloat16 if c.dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)

    def normal(*shape, std=0.02, mean=0.0):
        return torch.empty(shape, dtype=dt, device="cuda").normal_(mean, std, generator=g)

    d, hd, F = c.d_model, c.n_heads * c.head_dim, c.ffn_dim
    nq = (c.n_heads + 2 * c.n_kv_heads) * c.head_dim
    out_std = 0.02 / math.sqrt(2.0 * SHAPES[case["model"]][0])
    w = {"tok_emb": normal(c.vocab, d), "final_norm": normal(d, std=0.1, mean=1.0), "lm_head": normal(c.vocab, d)}
    for l in range(c.n_layers):
        w[f"layers.{l}.attn_norm"] = normal(d, std=0.1, mean=1.0)
        w[f"layers.{l}.w_qkv"] = normal(nq, d)
        w[f"layers.{l}.w_o"] = normal(d, hd, std=out_std)
        w[f"layers.{l}.mlp_norm"] = normal(d, std=0.1, mean=1.0)
        w[f"layers.{l}.w_gate_up"] = normal(2 * F, d)
        w[f"layers.{l}.w_down"] = normal(d, F, std=out_std)
    kv = torch.zeros((c.n_layers, 2, c.n_kv_heads, case["cap"], c.head_dim), dtype=dt, device="cuda")
    if case["ctx"]:
        kv[:, :, :, :case["ctx"]].normal_(0.0, 1.0, generator=g)
    n = case["rows"] + (1 if case["first"] else 0)
    tokens = np.random.default_rng([int(seed), 5]).integers(0, c.vocab, n).astype(np.int32)
    return w, kv, tokens


def prepare(case, seed):
    c = _config(case)
    w, kv, tokens = _inputs(case, seed)
    dw = binding.DeviceWeights(c, {})
    dw.tensors.update(w)
    torch.cuda.current_stream().synchronize()
    model = binding.Model(c, dw)
    if case["fp8"]:
        model.quantize_draft(_skip(case))
    logits = torch.empty((1 if case["first"] else case["rows"], c.vocab), dtype=torch.float32, device="cuda")
    new = kv[:, :, :, case["ctx"]:case["ctx"] + len(tokens)]  # the positions the call writes
    return {"model": model, "cache": model.cache(case["cap"], kv), "ctx": case["ctx"], "tokens": tokens,
            "first": case["first"], "skip": _skip(case) if _masked(case) else None, "logits": logits, "new": new}


def run(s):
    s["cache"].set_length(s["ctx"])
    if s["first"]:
        s["model"].forward(s["tokens"][:-1], s["cache"])
        s["model"].forward(s["tokens"][-1:], s["cache"], logits=s["logits"])
    else:
        s["model"].forward(s["tokens"], s["cache"], skip=s["skip"], logits=s["logits"])
    return {"logits": s["logits"], "kv": s["new"]}


# ----------------------------------------------------------------------------
# what a pass cannot do without


def work(case):
    c, z = _config(case), _skip(case)
    es = 2 if c.dtype == "bf16" else 4
    ws = 1 if case["fp8"] else es
    d, hd, F = c.d_model, c.n_heads * c.head_dim, c.ffn_dim
    kvd = c.n_kv_heads * c.head_dim
    attn_w, mlp_w, head_w = (2 * hd + 2 * kvd) * d, 3 * F * d, c.vocab * d
    n_attn, n_mlp = int((z[0::2] == 0).sum()), int((z[1::2] == 0).sum())
    n = case["rows"] + (1 if case["first"] else 0)
    n_head = 1 if case["first"] else n
    keys = sum(case["ctx"] + r + 1 for r in range(n))
    layer_w = n_attn * attn_w + n_mlp * mlp_w
    kv = 2 * kvd * es
    nbytes = layer_w * ws + head_w * es + n * d * es + n_attn * (case["ctx"] + n) * kv + n_head * c.vocab * 4
    if case["first"]:  # the first token is a second forward, which needs the prompt's keys
        nbytes += layer_w * ws + n_attn * n * kv
    flops = 2 * n * layer_w + 2 * n_head * head_w + n_attn * 4 * hd * keys
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times what a correct forward differs from exact() by.  float32: 2e-7.  bfloat16: keys and values are
    rounded to the cache's type, and a sum in another order rounds some of them the other way (one part in 256 of such
    a value); rows that attend to few cached keys carry that on most.  Measured: 1.3e-4 (verification over 512 keys or
    more), 9e-4 (prompts), 2.7e-3 (40 layers)."""
    if case["model"] == "tiny":
        return {"rel": 1e-6, "max": 1e-5}
    if case["first"]:
        return {"rel": 1.1e-2, "max": 8e-2}
    if case["rows"] > 16 or case["ctx"] < 256:
        return {"rel": 4e-3, "max": 4e-2}
    return {"rel": 5e-4, "max": 2e-2}


# ----------------------------------------------------------------------------
# the same forward in float64


def _rms(x, g):
    return g * (x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS))


def _fp8(w):
    """The value of each weight's E4M3 copy with one power-of-two scale per row (the smallest that fits 448)."""
    a = w.double()
    m, e = torch.frexp(a.abs().amax(1, keepdim=True))
    e = e - 9 + (m > 0.875).to(e.dtype)
    q = torch.ldexp(a, -e).float().to(torch.float8_e4m3fn).double()
    return torch.ldexp(q, e)


def _forward64(case, w, kv, tokens, pos, z, head):
    """Rows of tokens at pos.. over kv, which receives their keys and values; the logits of the rows if head."""
    c = _config(case)
    H, KVH, dh, F = c.n_heads, c.n_kv_heads, c.head_dim, c.ffn_dim
    M, half = len(tokens), dh // 2
    mat = _fp8 if case["fp8"] else (lambda t: t.double())
    h = w["tok_emb"][torch.from_numpy(tokens.astype(np.int64)).cuda()].double()
    theta = ROPE_BASE ** (-2.0 * torch.arange(half, dtype=torch.float64, device="cuda") / dh)
    ang = torch.arange(pos, pos + M, dtype=torch.float64, device="cuda")[:, None] * theta
    cos, sin = torch.cos(ang)[:, None], torch.sin(ang)[:, None]

    def rotate(x):
        a, b = x[..., :half], x[..., half:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)

    see = torch.arange(pos + M, device="cuda")[None, :] <= torch.arange(pos, pos + M, device="cuda")[:, None]
    for l in range(c.n_layers):
        p = f"layers.{l}."
        if not z[2 * l]:
            x = (_rms(h, w[p + "attn_norm"].double()) @ mat(w[p + "w_qkv"]).T).view(M, H + 2 * KVH, dh)
            q, k, v = rotate(x[:, :H]), rotate(x[:, H:H + KVH]), x[:, H + KVH:]
            kv[l, 0, :, pos:pos + M] = k.transpose(0, 1).to(kv.dtype)
            kv[l, 1, :, pos:pos + M] = v.transpose(0, 1).to(kv.dtype)
            o = torch.empty((M, H, dh), dtype=torch.float64, device="cuda")
            for i in range(H):
                kk, vv = (kv[l, j, i // (H // KVH), :pos + M].double() for j in (0, 1))
                s = (q[:, i] @ kk.T.contiguous()) / math.sqrt(dh)
                o[:, i] = torch.softmax(s.masked_fill(~see, -math.inf), -1) @ vv
            h = h + o.view(M, H * dh) @ mat(w[p + "w_o"]).T
        if not z[2 * l + 1]:
            x = _rms(h, w[p + "mlp_norm"].double()) @ mat(w[p + "w_gate_up"]).T
            h = h + (torch.nn.functional.silu(x[:, :F]) * x[:, F:]) @ mat(w[p + "w_down"]).T
    return _rms(h, w["final_norm"].double()) @ w["lm_head"].double().T if head else None


def exact(case, seed):
    w, kv, tokens = _inputs(case, seed)
    z = _skip(case)
    if case["first"]:
        _forward64(case, w, kv, tokens[:-1], case["ctx"], z, False)
        logits = _forward64(case, w, kv, tokens[-1:], case["ctx"] + len(tokens) - 1, z, True)
    else:
        logits = _forward64(case, w, kv, tokens, case["ctx"], z, True)
    return {"logits": logits, "kv": kv[:, :, :, case["ctx"]:case["ctx"] + len(tokens)].double()}
