"""The calls whose speed counts, through the library's public entry points.

A user of the library runs the MoE layer of a model (ms_forward) on decode
tokens and prompts, with the experts wholly in VRAM or split over VRAM and
host memory, in fp32, bf16 or 2-/4-bit codes; the attention block around it
(ms_dense, ms_rope_kv, ms_attention); and whole decoder tokens made of both.
Shapes are the ones of ``synth.py`` (tiny, Mixtral-8x7B, DeepSeek-V2-Lite,
Qwen3-30B-A3B, Mixtral with 2-bit codes); token counts are the benchmark's
(decode 1 and 16, prompts of 512 and 2048) and ragged ones between.

A few distinct expert weights are made per case and shared by the layer's
experts in host memory (ms_alias_expert); every expert cached in VRAM has its
own copy there, so a pass reads as many bytes as with distinct experts.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2509_08342_amd import moesplit as ms

# d_model, d_ff, experts, top-k, shared experts (of width d_ff), bits of an
# expert weight (32: fp32, 16: bf16, 4 or 2: affine codes), Zipf exponent of
# the router bias, distinct host weight sets
MODELS = {
    "tiny": dict(d=256, F=512, E=8, K=2, shared=0, bits=32, zipf=0.0, blobs=4),
    "mixtral": dict(d=4096, F=14336, E=8, K=2, shared=0, bits=16, zipf=0.0, blobs=1),
    "mixtral-q2": dict(d=4096, F=14336, E=8, K=2, shared=0, bits=2, zipf=0.0, blobs=1),
    "mixtral-q4": dict(d=4096, F=14336, E=8, K=2, shared=0, bits=4, zipf=0.0, blobs=1),
    "deepseek": dict(d=2048, F=1408, E=64, K=6, shared=2, bits=16, zipf=0.0, blobs=8),
    "qwen": dict(d=2048, F=768, E=128, K=8, shared=0, bits=16, zipf=1.1, blobs=16),
}
# largest token count of a case of each model
MOST_TOKENS = {"tiny": 64, "mixtral": 256, "mixtral-q2": 512, "mixtral-q4": 256, "deepseek": 512, "qwen": 2048}

# d_model, query heads, key/value heads, head width, most positions
HEADS = {
    "mixtral": dict(d=4096, Hq=32, Hkv=8, D=128, ctx=3360),
    "group8": dict(d=2048, Hq=32, Hkv=4, D=128, ctx=1360),
    "mha": dict(d=2048, Hq=16, Hkv=16, D=128, ctx=3360),
    "tiny": dict(d=256, Hq=4, Hkv=2, D=64, ctx=512),
}
ROPE_BASE = 1e6
VOCAB = 32000
WEIGHT_STD = 0.02
EPS = 1e-6


def listed():
    return [
        # the smallest layer, fp32: what a call costs when the weights cost nothing
        moe("tiny-f32-t4", "tiny", 4),
        # one decode token per layer, every expert in VRAM: the latency of a token
        moe("mixtral-decode", "mixtral", 1),
        moe("deepseek-decode", "deepseek", 1),
        moe("mixtral-q2-decode", "mixtral-q2", 1),
        # decode batches: the benchmark's 16 sequences, and a larger ragged batch
        moe("qwen-decode16", "qwen", 16),
        moe("deepseek-batch61", "deepseek", 61),
        # prompts
        moe("deepseek-prompt512", "deepseek", 512),
        moe("qwen-prompt2048", "qwen", 2048),
        moe("mixtral-q2-prompt512", "mixtral-q2", 512),
        # the attention block: a prompt, and one token deep in a context
        attention("attention-prompt2048", "mixtral", 2048, 0),
        attention("attention-decode1500", "mixtral", 1, 1500),
        # a whole decoder token over split experts (half of each expert and
        # two of eight tops per layer in VRAM, the rest streamed): attention,
        # MoE, prediction and prefetch, head, token
        dict(name="decoder-token-split", kind="token", model="mixtral-q2", heads="mixtral", layers=4, pos=600, r=0.5,
             cached=2),
    ]


def moe(name, model, T, r=1.0, cached=None, predict=True):
    c = dict(kind="moe", model=model, T=T, r=r, cached=MODELS[model]["E"] if cached is None else cached,
             predict=predict)
    return dict(name=name, **c) if name else c


def attention(name, heads, T, pos0):
    c = dict(kind="attention", heads=heads, T=T, pos0=pos0)
    return dict(name=name, **c) if name else c


def draw(rng):
    """A layer of one of the models at any token count of its range (one in
    six split over VRAM and host), or an attention block at any prompt length
    and position."""
    def log_uniform(lo, hi):
        return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))

    if rng.random() < 0.3:
        heads = rng.choice(["mixtral", "mixtral", "group8", "mha", "tiny"])
        ctx = HEADS[heads]["ctx"]
        T = 1 if rng.random() < 0.3 else log_uniform(2, min(2048, ctx))
        pos0 = rng.randint(0, ctx - T) if T <= 16 else rng.choice([0, 0, rng.randint(0, min(1024, ctx - T))])
        return attention(None, heads, T, pos0)
    model = rng.choice(["tiny", "mixtral", "mixtral-q2", "mixtral-q4", "deepseek", "deepseek", "qwen", "qwen"])
    T = log_uniform(1, MOST_TOKENS[model])
    E = MODELS[model]["E"]
    predict = rng.random() < 0.7
    if rng.random() < 1 / 6 and model != "mixtral":
        return moe(None, model, T, r=rng.choice([0.25, 0.5, 0.75, 0.9]), cached=rng.randint(E // 4, E),
                   predict=predict)
    return moe(None, model, T, predict=predict)


# ------------------------------------------------------------------ inputs

class Source:
    """Seeded draws on the GPU."""

    def __init__(self, seed, device="cuda"):
        self.gen = torch.Generator(device=device)
        self.gen.manual_seed(0x5EED0000 + seed)
        self.device = device

    def normal(self, *shape, std=1.0):
        x = torch.empty(shape, dtype=torch.float32, device=self.device)
        return x.normal_(0.0, std, generator=self.gen)

    def stored(self, bits, *shape, std=1.0):
        x = self.normal(*shape, std=std)
        return x if bits == 32 else x.to(torch.bfloat16)

    def integers(self, high, n):
        return torch.randint(0, high, (n,), dtype=torch.int32, device=self.device, generator=self.gen)


def host(x):
    """A device tensor's storage as a host array."""
    x = x.cpu()
    return x.view(torch.int16).numpy() if x.dtype == torch.bfloat16 else x.numpy()


def quantize(w, bits):
    """Affine codes of w [out][in] in groups of 64 along `in`, by rounding
    over each group's range: (codes uint8 [out][in], scale, zero fp16)."""
    g = w.view(w.shape[0], -1, 64)
    lo, hi = g.amin(2, keepdim=True), g.amax(2, keepdim=True)
    scale = ((hi - lo) / (2 ** bits - 1)).to(torch.float16)
    zero = (-lo / scale.float()).to(torch.float16)
    q = (g / scale.float() + zero.float()).round().clamp(0, 2 ** bits - 1).to(torch.uint8)
    return q.view(w.shape), scale.squeeze(2), zero.squeeze(2)


def packed(q, bits):
    """[out][in] codes as [out][in * bits / 8] bytes, low bits first."""
    per = 8 // bits
    out = torch.zeros(q.shape[0], q.shape[1] // per, dtype=torch.uint8, device=q.device)
    for j in range(per):
        out |= q[:, j::per] << (j * bits)
    return out


def make_expert(src, m):
    """One expert's tensors: three matrices, or three (codes, scale, zero)."""
    d, F, bits = m["d"], m["F"], m["bits"]
    if bits >= 16:
        return [src.stored(bits, *s, std=WEIGHT_STD) for s in ((d, F), (d, F), (F, d))]
    return [quantize(src.normal(*s, std=WEIGHT_STD), bits) for s in ((F, d), (F, d), (d, F))]


def make_layer(src, m):
    """Router [d][E] and its bias of one layer."""
    router = src.stored(16 if m["bits"] < 32 else 32, m["d"], m["E"], std=WEIGHT_STD)
    bias = None
    if m["zipf"]:
        rank = torch.argsort(torch.rand(m["E"], device=src.device, generator=src.gen))
        bias = (-m["zipf"] * torch.log1p(rank.double())).float()
    return router, bias


def moe_inputs(case, seed, layers=1):
    """(hidden rows, [router, bias] per layer, experts, shared experts)."""
    m = MODELS[case["model"]]
    src = Source(seed)
    rows = src.stored(16 if m["bits"] < 32 else 32, case.get("T", 1), m["d"])
    routers = [make_layer(src, m) for _ in range(layers)]
    experts = [make_expert(src, m) for _ in range(m["blobs"])]
    shared = [make_expert(src, m) for _ in range(m["shared"])]
    return src, rows, routers, experts, shared


def attention_inputs(case, seed, layers=1):
    """Attention weights of `layers` layers and their caches of past keys and values."""
    a = HEADS[case["heads"]]
    src = Source(seed + (1 << 20))
    n_qkv = (a["Hq"] + 2 * a["Hkv"]) * a["D"]
    w_qkv = [src.stored(16, n_qkv, a["d"], std=WEIGHT_STD) for _ in range(layers)]
    w_o = [src.stored(16, a["d"], a["Hq"] * a["D"], std=WEIGHT_STD) for _ in range(layers)]
    past = case.get("pos0", case.get("pos", 0))
    kc = torch.zeros(layers, a["Hkv"], a["ctx"], a["D"], dtype=torch.bfloat16, device="cuda")
    vc = torch.zeros_like(kc)
    for c in (kc, vc):  # rows already in the context, of the size the projections give
        c[:, :, :past] = src.normal(layers, a["Hkv"], past, a["D"], std=WEIGHT_STD * math.sqrt(a["d"])).to(c.dtype)
    return src, w_qkv, w_o, kc, vc


class Layers:
    """A context with its pool, experts set, tops cached: what a program keeps."""

    def __init__(self, case, routers, experts, shared, max_tokens, cached):
        m = MODELS[case["model"]]
        L = len(routers)
        f32 = m["bits"] == 32
        self.desc = ms.ms_model_desc(L, m["d"], m["F"], m["E"], m["K"], m["shared"], m["F"] if m["shared"] else 0,
                                     ms.MS_F32 if f32 else ms.MS_BF16, 1, max_tokens, 0, 0,
                                     m["bits"] if m["bits"] < 16 else 0)
        sizes = ms.ms_query_sizes(self.desc)
        top = ms.ms_split_plan(self.desc, 0, case["r"])[1]
        budget = max(top, 1) * cached
        pool_bytes = sizes.fixed_pool_bytes + budget * L
        self.pool = torch.empty(pool_bytes, dtype=torch.uint8, device="cuda")
        self.ctx = ms.ms_create(self.desc, self.pool, pool_bytes, len(experts))
        for l, (router, bias) in enumerate(routers):
            ms.ms_set_router(self.ctx, l, host(router), None if bias is None else host(bias))
        for e, ex in enumerate(experts):
            if m["bits"] >= 16:
                ms.ms_set_expert(self.ctx, 0, e, *[host(w) for w in ex])
            else:
                ms.ms_set_expert_q(self.ctx, 0, e, [host(packed(q, m["bits"])) for q, _, _ in ex],
                                   [host(torch.stack([s, z], 2)).view(np.uint16) for _, s, z in ex])
        for l in range(L):
            for e in range(m["E"]):
                if l or e >= len(experts):
                    ms.ms_alias_expert(self.ctx, l, e, 0, e % len(experts))
            for i, ex in enumerate(shared):
                ms.ms_set_shared_expert(self.ctx, l, i, *[host(w) for w in ex])
        ms.ms_configure(self.ctx, [budget] * L, [case["r"]] * L)
        for l in range(L):
            for e in range(cached):
                ms.ms_load_top(self.ctx, l, e)
        ms.ms_sync(self.ctx)

    def __del__(self):
        if getattr(self, "ctx", None) is not None:
            ms.ms_sync(self.ctx)
            ms.ms_destroy(self.ctx)
            self.ctx = None


def prepare(case, seed):
    st = dict(case=case)
    kind = case["kind"]
    f32, bf16, i32 = torch.float32, torch.bfloat16, torch.int32

    def empty(dtype, *shape):
        return torch.empty(shape, dtype=dtype, device="cuda")

    if kind in ("moe", "token"):
        m = MODELS[case["model"]]
        T = case.get("T", 1)
        _, rows, routers, experts, shared = moe_inputs(case, seed, case.get("layers", 1))
        st.update(h=rows, layers=Layers(case, routers, experts, shared, T, case["cached"]), y=empty(f32, T, m["d"]),
                  idx=empty(i32, T, m["K"]), w=empty(f32, T, m["K"]))
    if kind in ("attention", "token"):
        a = HEADS[case["heads"]]
        T = case.get("T", 1)
        src, w_qkv, w_o, kc, vc = attention_inputs(case, seed, case.get("layers", 1))
        st.update(w_qkv=w_qkv, w_o=w_o, kc=kc, vc=vc, qkv=empty(f32, T, w_qkv[0].shape[0]),
                  q=empty(bf16, T, a["Hq"], a["D"]), o=empty(bf16, T, a["Hq"] * a["D"]), att=empty(f32, T, a["d"]))
        if kind == "attention":
            st["x"] = src.stored(16, T, a["d"])
        else:
            st.update(head=src.stored(16, VOCAB, a["d"], std=WEIGHT_STD), embed=src.stored(16, VOCAB, a["d"]),
                      ids=src.integers(VOCAB, 1), x=[empty(bf16, 1, a["d"]) for _ in range(3)],
                      hh=empty(bf16, 1, a["d"]), logits=empty(f32, 1, VOCAB), token=empty(i32, 1))
    return st


# -------------------------------------------------------------------- runs

def attention_block(st, a, layer, x, T, pos0, stream):
    n_qkv = st["qkv"].shape[1]
    ms.ms_dense(x, st["w_qkv"][layer], T, a["d"], n_qkv, st["qkv"], None, stream)
    ms.ms_rope_kv(st["qkv"], T, a["Hq"], a["Hkv"], a["D"], pos0, ROPE_BASE, st["q"], st["kc"][layer], st["vc"][layer],
                  a["ctx"], stream)
    ms.ms_attention(st["q"], st["kc"][layer], st["vc"][layer], T, a["Hq"], a["Hkv"], a["D"], pos0, a["ctx"], st["o"],
                    stream)
    ms.ms_dense(st["o"], st["w_o"][layer], T, a["Hq"] * a["D"], a["d"], st["att"], None, stream)


def run(st):
    case = st["case"]
    stream = torch.cuda.current_stream()
    if case["kind"] == "moe":
        ms.ms_forward(st["layers"].ctx, 0, st["h"], case["T"], st["y"], st["idx"], st["w"],
                      ms.MS_FWD_PREDICT_NEXT if case["predict"] else 0, stream)
        return dict(y=st["y"], idx=st["idx"], w=st["w"])
    a = HEADS[case["heads"]]
    if case["kind"] == "attention":
        T, pos0 = case["T"], case["pos0"]
        attention_block(st, a, 0, st["x"], T, pos0, stream)
        return dict(att=st["att"], o=st["o"], k=st["kc"][0, :, pos0:pos0 + T], v=st["vc"][0, :, pos0:pos0 + T])
    ctx, d = st["layers"].ctx, a["d"]
    src = st["x"][2]
    ms.ms_embed(st["ids"], st["embed"], VOCAB, 1, d, src, stream)
    for l in range(case["layers"]):
        attention_block(st, a, l, src, 1, case["pos"], stream)
        ms.ms_residual_norm(ctx, src, st["att"], 1, st["hh"], stream)
        ms.ms_forward(ctx, l, st["hh"], 1, st["y"], st["idx"], st["w"], ms.MS_FWD_PREDICT_NEXT, stream)
        ms.ms_residual_norm(ctx, st["hh"], st["y"], 1, st["x"][l % 2], stream)
        src = st["x"][l % 2]
    ms.ms_dense(src, st["head"], 1, d, VOCAB, st["logits"], None, stream)
    ms.ms_argmax(st["logits"], 1, VOCAB, st["token"], stream)
    return dict(logits=st["logits"], token=st["token"], x=src, k=st["kc"][:, :, case["pos"]],
                v=st["vc"][:, :, case["pos"]])


# ------------------------------------------------------- work and tolerance

def expert_bytes(m):
    n = 3 * m["d"] * m["F"]
    return n * m["bits"] // 8 + (n // 64 * 4 if m["bits"] < 16 else 0)


def active_experts(m, T):
    """Distinct experts that T tokens select, for random rows and routers."""
    rng = np.random.RandomState(7)
    std = WEIGHT_STD * math.sqrt(m["d"])
    lg = rng.standard_normal((T, m["E"])) * std - m["zipf"] * np.log1p(np.arange(m["E"]))
    return len(np.unique(np.argpartition(-lg, m["K"] - 1, axis=1)[:, :m["K"]]))


def moe_work(m, T):
    elem = 4 if m["bits"] == 32 else 2
    d, F, E, K = m["d"], m["F"], m["E"], m["K"]
    n_bytes = ((active_experts(m, T) + m["shared"]) * expert_bytes(m) + d * E * elem + T * d * (elem + 4) + T * K * 8)
    flops = 6.0 * T * (K + m["shared"]) * d * F + 2.0 * T * d * E
    return n_bytes, flops


def attention_work(a, T, pos0):
    d, Hq, Hkv, D = a["d"], a["Hq"], a["Hkv"], a["D"]
    w = (Hq + 2 * Hkv) * D * d + d * Hq * D
    pairs = T * pos0 + T * (T + 1) / 2
    return 2 * w + T * d * (2 + 4) + 4 * Hkv * D * (pos0 + T) + 2 * T * Hq * D, 2.0 * T * w + 4.0 * Hq * D * pairs


def work(case):
    if case["kind"] == "moe":
        b, f = moe_work(MODELS[case["model"]], case["T"])
    elif case["kind"] == "attention":
        b, f = attention_work(HEADS[case["heads"]], case["T"], case["pos0"])
    else:
        a = HEADS[case["heads"]]
        bm, fm = moe_work(MODELS[case["model"]], 1)
        ba, fa = attention_work(a, 1, case["pos"])
        b = case["layers"] * (bm + ba) + 2 * VOCAB * a["d"] + 4 * VOCAB
        f = case["layers"] * (fm + fa) + 2.0 * VOCAB * a["d"]
    return dict(bytes=float(b), flops=float(f))


def tolerance(case):
    """About four times the distance from exact(): fp32 sums with products of
    at least 16 mantissa bits (2.4e-6 seen), bf16 SwiGLU values on their way
    into the down projection (1.7e-3), bf16 queries, keys, values and
    attention rows (4e-3 where a few keys dominate a row), and for a whole
    token the same through four layers of bf16 activations (1.2e-2)."""
    if case["kind"] == "moe":
        m = MODELS[case["model"]]
        rounded = m["bits"] < 16 or (m["bits"] == 16 and case["T"] * m["K"] >= 8 * m["E"])
        return dict(rel=7e-3) if rounded else dict(rel=1e-5)
    return dict(rel=1.5e-2) if case["kind"] == "attention" else dict(rel=3e-2)


# ------------------------------------------------------------------- exact

def matrices64(m, ex):
    """An expert's (gate [d][F], up [d][F], down [F][d]) in 64 bits."""
    if m["bits"] >= 16:
        return [w.double() for w in ex]
    out = []
    for q, s, z in ex:
        g = q.view(q.shape[0], -1, 64).double()
        out.append(((g - z.double()[:, :, None]) * s.double()[:, :, None]).view(q.shape).t())
    return out


def exact_moe(m, h, router, bias, experts, shared):
    lg = h @ router.double()
    if bias is not None:
        lg = lg + bias.double()
    top, idx = torch.topk(lg, m["K"], dim=1)
    w = torch.softmax(top, 1)
    y = torch.zeros_like(h)
    for b, ex in enumerate(experts):  # expert e has the weights of set e % blobs
        t, k = torch.nonzero(idx % len(experts) == b, as_tuple=True)
        if len(t):
            g, u, dn = matrices64(m, ex)
            x = h[t]
            y.index_add_(0, t, w[t, k][:, None] * ((torch.nn.functional.silu(x @ g) * (x @ u)) @ dn))
    for ex in shared:
        g, u, dn = matrices64(m, ex)
        y += (torch.nn.functional.silu(h @ g) * (h @ u)) @ dn
    return y, idx, w


def exact_attention(a, x, w_qkv, w_o, kc, vc, pos0):
    T, Hq, Hkv, D = x.shape[0], a["Hq"], a["Hkv"], a["D"]
    qkv = (x @ w_qkv.double().t()).view(T, Hq + 2 * Hkv, D)
    i = torch.arange(D // 2, dtype=torch.float64, device=x.device)
    ang = torch.arange(pos0, pos0 + T, dtype=torch.float64, device=x.device)[:, None] * ROPE_BASE ** (-2 * i / D)
    c, s = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    x1, x2 = qkv[..., :D // 2], qkv[..., D // 2:]
    turned = torch.cat([x1 * c - x2 * s, x2 * c + x1 * s], 2)
    q, k, v = turned[:, :Hq], turned[:, Hq:Hq + Hkv], qkv[:, Hq + Hkv:]
    k, v = k.transpose(0, 1), v.transpose(0, 1)
    keys = torch.cat([kc[:, :pos0].double(), k], 1)
    vals = torch.cat([vc[:, :pos0].double(), v], 1)
    o = torch.empty(T, Hq, D, dtype=torch.float64, device=x.device)
    n = pos0 + T
    later = torch.arange(n, device=x.device)[None, :] > torch.arange(pos0, n, device=x.device)[:, None]
    for hd in range(Hq):
        sc = (q[:, hd] @ keys[hd * Hkv // Hq].t()) / math.sqrt(D)
        o[:, hd] = torch.softmax(sc.masked_fill(later, -math.inf), 1) @ vals[hd * Hkv // Hq]
    o = o.view(T, Hq * D)
    return o @ w_o.double().t(), o, k, v


def norm64(x):
    return x / torch.sqrt((x * x).mean(1, keepdim=True) + EPS)


def exact(case, seed):
    if case["kind"] == "moe":
        m = MODELS[case["model"]]
        _, rows, routers, experts, shared = moe_inputs(case, seed)
        y, idx, w = exact_moe(m, rows.double(), *routers[0], experts, shared)
        return dict(y=y, idx=None, w=w)
    a = HEADS[case["heads"]]
    src, w_qkv, w_o, kc, vc = attention_inputs(case, seed, case.get("layers", 1))
    if case["kind"] == "attention":
        x = src.stored(16, case["T"], a["d"])
        att, o, k, v = exact_attention(a, x.double(), w_qkv[0], w_o[0], kc[0], vc[0], case["pos0"])
        return dict(att=att, o=o, k=k, v=v)
    m = MODELS[case["model"]]
    head, embed = src.stored(16, VOCAB, a["d"], std=WEIGHT_STD), src.stored(16, VOCAB, a["d"])
    ids = src.integers(VOCAB, 1)
    _, _, routers, experts, shared = moe_inputs(case, seed, case["layers"])
    x, ks, vs = embed[ids.long()].double(), [], []
    for l in range(case["layers"]):
        att, _, k, v = exact_attention(a, x, w_qkv[l], w_o[l], kc[l], vc[l], case["pos"])
        h = norm64(x + att)
        x = norm64(h + exact_moe(m, h, *routers[l], experts, shared)[0])
        ks.append(k[:, 0])
        vs.append(v[:, 0])
    return dict(logits=x @ head.double().t(), token=None, x=x, k=torch.stack(ks), v=torch.stack(vs))
