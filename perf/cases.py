"""The measured work of this framework: what its users have it do, through the
package's public entry points, over the sizes it is used at.

Shapes are those of workloads/configs.py: the two-layer float32 decoder of the
tests, the LLaVA-1.5-7B and -13B shapes and the grouped-query 7B shape with a
wide FFN.  Decoder stacks are shortened to a few layers where a whole one would
only repeat the same launches; the batch-1 prefill runs all 32.

Kinds of case:
  prefill     svl_prefill, or svl_prefill_cache (cache=True), of a batch
  decode      svl_decode_step: one new token per sample on the cached keys
  train       svl_train_step: forward and backward of the masked decoder
  controlled  svl_prefill_controlled: the compute controller in the loop
  select      svl_select_tokens alone: selection and packing
"""
import math
import random

import numpy as np
import torch

import paper_2607_20357_amd as svl

SHAPES = {
    "tiny": dict(d_model=256, n_heads=4, n_kv_heads=4, head_dim=64, d_ffn=688),
    "llava7b": dict(d_model=4096, n_heads=32, n_kv_heads=32, head_dim=128, d_ffn=11008),
    "gqa7b": dict(d_model=3584, n_heads=28, n_kv_heads=4, head_dim=128, d_ffn=18944),
    "llava13b": dict(d_model=5120, n_heads=40, n_kv_heads=40, head_dim=128, d_ffn=13824),
}
GROUPS = 4
EPS, THETA = 1e-6, 10000.0
TAU_TOK, TAU_COMP = 0.7, 1.3
PE_DIM, PE_SCALE, PE_BASE = 256, 1000.0, 10000.0


def _prefill(name, shape, layers, n_vision, n_text, keep, groups, skipped, compute="f16",
             cache=False):
    """keep, groups, skipped: per sample, as comma-separated texts: keep ratio,
    head groups (of 4) on in every executed layer, layers skipped."""
    return dict(name=name, kind="prefill", shape=shape, layers=layers, n_vision=n_vision,
                n_text=n_text, keep=keep, groups=groups, skipped=skipped, compute=compute,
                cache=cache)


def listed():
    return [
        # the smallest call, float32 storage and arithmetic: launches and host time
        _prefill("prefill_tiny_f32", "tiny", 2, 64, 16, "0.5", "3", "0"),
        # one image and a question, a whole 32-layer stack: the serving latency
        # that the framework is quoted on
        _prefill("prefill_7b_b1", "llava7b", 32, 576, 64, "0.25", "3", "8"),
        # the same with bfloat16 activations, filling the cache for the decode
        # that follows; odd lengths
        _prefill("prefill_7b_b1_bf16_cache", "llava7b", 8, 577, 61, "0.5", "3", "2", "bf16", True),
        # a serving batch of requests at different budgets
        _prefill("prefill_7b_b8", "llava7b", 4, 576, 64, "1.0,0.5,0.25,0.11,0.5,1.0,0.25,0.5",
                 "4,3,2,3,4,2,3,4", "0,1,0,1,0,0,1,0"),
        # high-resolution crops, grouped-query attention, wide FFN
        _prefill("prefill_gqa7b_b2", "gqa7b", 4, 2880, 128, "0.2,0.2", "3,3", "1,0"),
        # video tokens, 13B shape, half of the groups
        _prefill("prefill_13b_video_b4", "llava13b", 4, 3136, 64, "0.1,0.1,0.1,0.1", "2,2,2,2",
                 "1,1,0,1"),
        # one new token of one request
        dict(name="decode_7b_b1", kind="decode", shape="llava7b", layers=8, cached="208",
             groups="3", skipped="2", compute="f16"),
        # one new token of each of eight requests
        dict(name="decode_7b_b8", kind="decode", shape="llava7b", layers=4,
             cached="640,352,208,127,352,640,208,352", groups="4,3,2,3,4,2,3,4",
             skipped="0,1,0,1,0,0,1,0", compute="f16"),
        # a training step's decoder, one sample at full length, bf16 weights
        dict(name="train_7b_b1", kind="train", shape="llava7b", layers=2, prefix=1, batch=1,
             n_vision=576, n_text=64, dtype="bf16"),
        # the smallest training step, float32 weights
        dict(name="train_tiny_f32", kind="train", shape="tiny", layers=2, prefix=1, batch=2,
             n_vision=64, n_text=16, dtype="f32"),
        # budget token, controller, projection to the budget, second half of the stack
        dict(name="controlled_7b_b1", kind="controlled", shape="llava7b", layers=8, prefix=4,
             batch=1, n_vision=576, n_text=64, budget=0.25, positive=0.26, compute="f16"),
        # packing a large batch ahead of a pipeline: memory traffic
        dict(name="select_b64", kind="select", shape="llava7b", batch=64, n_vision=576, n_text=64,
             keep=0.25),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def texts(values):
        return ",".join(str(v) for v in values)

    kind = rng.choice(["prefill", "prefill", "prefill", "decode", "decode", "train", "train",
                       "controlled", "select"])
    big = rng.choice(["llava7b", "llava7b", "gqa7b", "llava13b"])
    if kind == "prefill":
        batch = rng.choice([1, 1, 2, 3, 4, 6, 8])
        layers = rng.choice([1, 2, 3])
        n = log_int(64, 3136)
        ratios = [r for r in (1.0, 0.5, 0.25, 0.2, 0.11, 0.1) if r * n * batch <= 2048] or [0.1]
        return dict(kind="prefill", shape=big, layers=layers, n_vision=n, n_text=log_int(8, 160),
                    keep=texts(rng.choice(ratios) for _ in range(batch)),
                    groups=texts(rng.choice([2, 3, 4]) for _ in range(batch)),
                    skipped=texts(rng.choice([0, 0, 1]) if layers > 1 else 0 for _ in range(batch)),
                    compute=rng.choice(["f16", "f16", "bf16"]), cache=rng.random() < 0.3)
    if kind == "decode":
        batch = rng.choice([1, 1, 2, 4, 8])
        layers = rng.choice([2, 3, 4])
        return dict(kind="decode", shape=big, layers=layers,
                    cached=texts(log_int(24, 1500) for _ in range(batch)),
                    groups=texts(rng.choice([2, 3, 4]) for _ in range(batch)),
                    skipped=texts(rng.choice([0, 0, 1]) for _ in range(batch)),
                    compute=rng.choice(["f16", "f16", "bf16"]))
    if kind == "train":
        shape, dtype = rng.choice([("tiny", "f32"), (big, "bf16"), (big, "bf16")])
        n, t = log_int(48, 576), log_int(8, 64)
        batch = rng.choice([1, 2, 3]) if shape == "tiny" or n < 250 else 1
        return dict(kind="train", shape=shape, layers=rng.choice([1, 2]) if shape == "tiny" else 1,
                    prefix=rng.choice([0, 1]), batch=batch, n_vision=n, n_text=t, dtype=dtype)
    if kind == "controlled":
        return dict(kind="controlled", shape=big, layers=4, prefix=2, batch=rng.choice([1, 1, 2]),
                    n_vision=log_int(144, 1152), n_text=log_int(16, 96),
                    budget=rng.choice([0.25, 0.5, 1.0]), positive=rng.choice([0.26, 0.5]),
                    compute="f16")
    return dict(kind="select", shape=big, batch=log_int(1, 64), n_vision=log_int(196, 3136),
                n_text=log_int(8, 128), keep=rng.choice([0.11, 0.25, 0.5]))


# ------------------------------------------------------------------ sizes of a case
def _ints(text):
    return [int(v) for v in str(text).split(",")]


def _keep_counts(case):
    if case["kind"] == "select":
        return [int(math.floor(case["keep"] * case["n_vision"] + 0.5))] * case["batch"]
    return [int(math.floor(float(r) * case["n_vision"] + 0.5)) for r in case["keep"].split(",")]


def _dtype(case):
    if "dtype" in case:
        return case["dtype"]
    return "f32" if case["shape"] == "tiny" else "bf16"


def _config(case):
    return svl.make_config(None, n_layers=case.get("layers", 1), n_groups=GROUPS, rms_eps=EPS,
                           rope_theta=THETA, dtype=_dtype(case), compute=case.get("compute", "f16"),
                           **SHAPES[case["shape"]])


# ------------------------------------------------------------------ inputs
class _Draws:
    """Seeded tensors on the GPU: one generator per state, used in a fixed order."""

    def __init__(self, seed):
        self.dev = torch.device("cuda")
        self.g = torch.Generator(device=self.dev)
        self.g.manual_seed(int(seed) * 7919 + 17)
        self.rng = random.Random(int(seed) * 104729 + 5)

    def normal(self, shape, dtype=torch.float32, mean=0.0, std=1.0):
        return torch.empty(shape, dtype=dtype, device=self.dev).normal_(mean, std, generator=self.g)

    def uniform(self, shape):
        return torch.empty(shape, dtype=torch.float32, device=self.dev).uniform_(1e-6, 1 - 1e-6,
                                                                                  generator=self.g)


def _layers(case, dr):
    s = SHAPES[case["shape"]]
    D, F = s["d_model"], s["d_ffn"]
    Aw, Kw = s["n_heads"] * s["head_dim"], s["n_kv_heads"] * s["head_dim"]
    dt = torch.bfloat16 if _dtype(case) == "bf16" else torch.float32
    dims = dict(wq=(Aw, D), wk=(Kw, D), wv=(Kw, D), wo=(D, Aw), w_gate=(F, D), w_up=(F, D),
                w_down=(D, F))
    out = []
    for _ in range(case["layers"]):
        w = {n: dr.normal(shape, dt, 0.0, 0.02) for n, shape in dims.items()}
        w["attn_norm"] = dr.normal((D,), torch.float32, 1.0, 0.02).to(dt)
        w["ffn_norm"] = dr.normal((D,), torch.float32, 1.0, 0.02).to(dt)
        out.append(w)
    return out


def _masks(case, dr):
    """Layer, head and FFN-slice masks: each sample skips `skipped` layers of
    the second half of its stack and runs `groups` of its 4 head groups."""
    L, A = case["layers"], SHAPES[case["shape"]]["n_heads"]
    groups, skipped = _ints(case["groups"]), _ints(case["skipped"])
    B = len(groups)
    layer_on = np.ones((B, L), np.uint8)
    group_on = np.zeros((B, L, GROUPS), np.uint8)
    for b in range(B):
        half = list(range(L // 2, L))
        for l in dr.rng.sample(half, min(skipped[b], len(half))):
            layer_on[b, l] = 0
        for l in range(L):
            group_on[b, l, dr.rng.sample(range(GROUPS), groups[b])] = 1
    return layer_on, np.repeat(group_on, A // GROUPS, axis=2), group_on


def _hidden(case, dr, batch):
    dt = torch.bfloat16 if _dtype(case) == "bf16" else torch.float32
    D = SHAPES[case["shape"]]["d_model"]
    return (dr.normal((batch, case["n_vision"], D), dt), dr.normal((batch, case["n_text"], D), dt))


def _controller(case, dr):
    D = SHAPES[case["shape"]]["d_model"]
    n = (case["layers"] - case["prefix"]) * GROUPS
    bf = torch.bfloat16
    t = dict(llm_w1=dr.normal((D, PE_DIM), bf, 0.0, (2.0 / PE_DIM) ** 0.5),
             llm_w2=dr.normal((D, D), bf, 0.0, (1.0 / D) ** 0.5),
             kap_w1=dr.normal((D, PE_DIM), bf, 0.0, (2.0 / PE_DIM) ** 0.5),
             kap_w2=dr.normal((D, D), bf, 0.0, (1.0 / D) ** 0.5),
             gate_w=dr.normal((n, D), bf, 0.0, 0.002 / D ** 0.5))
    for name in ("llm_b1", "llm_b2", "kap_b1", "kap_b2"):
        t[name] = dr.normal((D,), bf, 0.0, 0.1)
    # each unit's bias fixes its decision and keeps every pair of logits apart
    ranks = dr.rng.sample(range(n), n)
    sign = [1.0 if r % 4 else -1.0 for r in ranks]
    t["gate_b"] = torch.tensor([s * (0.5 + 0.1 * r) for s, r in zip(sign, ranks)]).to("cuda", bf)
    return t


def prepare(case, seed):
    dr = _Draws(seed)
    kind = case["kind"]
    cfg = _config(case)
    s = SHAPES[case["shape"]]
    D = s["d_model"]
    st = dict(case=case, cfg=cfg)
    if kind == "select":
        B, N, T = case["batch"], case["n_vision"], case["n_text"]
        st["vision"], st["text"] = _hidden(case, dr, B)
        st["scores"] = torch.exp(dr.normal((B, N)))
        st["keep"] = np.array(_keep_counts(case), np.int32)
        R = int(st["keep"].sum()) + B * T
        st["kept"] = torch.empty((B, N), dtype=torch.int32, device="cuda")
        st["resid"] = torch.empty((R, D), dtype=torch.float32, device="cuda")
        st["ws"] = svl.alloc_workspace(cfg, B, R)
        return st
    weights = _layers(case, dr)
    st["weights"] = weights
    st["table"] = svl.LayerTable(weights)
    if kind == "prefill":
        keep = _keep_counts(case)
        B, N, T = len(keep), case["n_vision"], case["n_text"]
        st["vision"], st["text"] = _hidden(case, dr, B)
        st["scores"] = torch.exp(dr.normal((B, N)))
        st["keep"] = np.array(keep, np.int32)
        st["masks"] = _masks(case, dr)
        R = sum(keep) + B * T
        st["kept"] = torch.empty((B, N), dtype=torch.int32, device="cuda")
        st["resid"] = torch.empty((R, D), dtype=torch.float32, device="cuda")
        st["ws"] = svl.alloc_workspace(cfg, B, R)
        if case["cache"]:
            st["max_len"] = max(keep) + T + 64
            st["kv"] = svl.alloc_kv_cache(cfg, B, st["max_len"]).zero_()
    elif kind == "decode":
        lens = _ints(case["cached"])
        B = len(lens)
        st["max_len"] = (max(lens) // 128 + 1) * 128
        st["lens"] = np.array(lens, np.int32)
        st["masks"] = _masks(case, dr)
        st["emb"] = dr.normal((B, D))
        st["x"] = torch.empty_like(st["emb"])
        act = torch.float16 if case["compute"] == "f16" else torch.bfloat16
        kv = svl.alloc_kv_cache(cfg, B, st["max_len"])
        kv.view(act).normal_(0.0, 1.0, generator=dr.g)
        st["kv"] = kv
        st["ws"] = svl.alloc_decode_workspace(cfg, B, st["max_len"])
    elif kind == "train":
        B, N, T = case["batch"], case["n_vision"], case["n_text"]
        nl = (case["layers"] - case["prefix"]) * GROUPS
        st["params"] = svl.svl_train_params(TAU_TOK, TAU_COMP, case["prefix"], GROUPS)
        st["vision"], st["text"] = _hidden(case, dr, B)
        st["z"] = dr.normal((B, N), mean=0.3, std=1.5)
        st["g"] = dr.normal((B, nl), mean=0.6, std=1.5)
        u, v = dr.uniform((B, N)), dr.uniform((B, nl))
        st["zn"] = torch.log(u) - torch.log1p(-u)
        st["gn"] = torch.log(v) - torch.log1p(-v)
        st["grad"] = dr.normal((B, N + T, D))
        st["ws"] = svl.alloc_train_workspace(cfg, st["params"], B, N, T)
    else:
        B, N, T = case["batch"], case["n_vision"], case["n_text"]
        st["vision"], st["text"] = _hidden(case, dr, B)
        # a fixed share of positive logits, at places drawn for each sample
        z = dr.normal((B, N)).abs() + 0.01
        order = torch.argsort(dr.uniform((B, N)), dim=1)
        z.scatter_(1, order[:, int(case["positive"] * N):],
                   -z.gather(1, order[:, int(case["positive"] * N):]))
        st["z"] = z
        st["ctrl"] = svl.Controller(case["prefix"], GROUPS, PE_DIM, D, PE_SCALE, PE_BASE,
                                    _controller(case, dr))
        st["kept"] = torch.empty((B, N), dtype=torch.int32, device="cuda")
        st["resid"] = torch.zeros((B * (N + T + 1), D), dtype=torch.float32, device="cuda")
        st["ws"] = svl.alloc_controlled_workspace(cfg, st["ctrl"], B, N, T)
    return st


# ------------------------------------------------------------------ one pass
def run(st):
    case, cfg = st["case"], st["cfg"]
    kind = case["kind"]
    if kind == "select":
        svl.svl_select_tokens(cfg, st["keep"], st["scores"], st["vision"], st["text"], st["kept"],
                              st["resid"], st["ws"])
        return {"kept": st["kept"], "resid": st["resid"]}
    if kind == "prefill":
        lm, hm, fm = st["masks"]
        if not case["cache"]:
            svl.svl_prefill(cfg, st["table"], st["keep"], st["scores"], st["vision"], st["text"],
                            lm, hm, fm, st["kept"], st["resid"], st["ws"], want_flops=False)
            return {"kept": st["kept"], "resid": st["resid"]}
        svl.svl_prefill_cache(cfg, st["table"], st["keep"], st["scores"], st["vision"], st["text"],
                              lm, hm, fm, st["kept"], st["resid"], st["kv"], st["max_len"], st["ws"])
        return {"kept": st["kept"], "resid": st["resid"], "cache": _cache_view(case, st["kv"])}
    if kind == "decode":
        lm, hm, fm = st["masks"]
        st["x"].copy_(st["emb"])   # the new tokens' embeddings
        svl.svl_decode_step(cfg, st["table"], st["x"], st["lens"], lm, hm, fm, st["kv"],
                            st["max_len"], st["ws"])
        return {"x": st["x"], "cache": _cache_view(case, st["kv"])}
    if kind == "train":
        return svl.svl_train_step(cfg, st["table"], st["params"], st["z"], st["g"], st["vision"],
                                  st["text"], st["grad"], st["ws"], token_noise=st["zn"],
                                  gate_noise=st["gn"])
    out = svl.svl_prefill_controlled(cfg, st["table"], st["ctrl"], st["z"], st["vision"],
                                     st["text"], case["budget"], 0, st["kept"], st["resid"],
                                     st["ws"], want_flops=False)
    rows = int(out["cu_seqlens"][-1])
    return {"kept": st["kept"], "resid": st["resid"][:rows], "keep": out["keep"],
            "layer_mask": out["layer_mask"], "head_mask": out["head_mask"],
            "ffn_mask": out["ffn_mask"], "gate_logits": out["gate_logits"]}


def _cache_view(case, kv):
    return kv.view(torch.float16 if case["compute"] == "f16" else torch.bfloat16)


# ------------------------------------------------------------------ what a pass cannot do without
def _layer_cost(s, rows_on, es):
    """(flops, weight bytes) of one layer for [(rows, groups on)] of the samples
    that run it; weights that several samples use are read once."""
    D, A, KV, d, F = (s[k] for k in ("d_model", "n_heads", "n_kv_heads", "head_dim", "d_ffn"))
    w = (2 * A * d + 2 * KV * d + 3 * F) * D
    flops, unused = 0.0, 1.0
    for S, g in rows_on:
        flops += 2.0 * S * w * g / GROUPS + 2.0 * A * g / GROUPS * d * S * (S + 1)
        unused *= 1.0 - g / GROUPS
    return flops, w * es * (1.0 - unused)


def work(case):
    s = SHAPES[case["shape"]]
    D, A, KV, d, F = (s[k] for k in ("d_model", "n_heads", "n_kv_heads", "head_dim", "d_ffn"))
    es = 2 if _dtype(case) == "bf16" else 4
    kind = case["kind"]
    flops = nbytes = 0.0
    if kind in ("select", "prefill"):
        keep = _keep_counts(case)
        B, N, T = len(keep), case["n_vision"], case["n_text"]
        R = sum(keep) + B * T
        nbytes = B * N * 8 + R * D * (es + 4)
        if kind == "prefill":
            groups, skipped = _ints(case["groups"]), _ints(case["skipped"])
            L = case["layers"]
            for l in range(L):
                on = [(keep[b] + T, groups[b]) for b in range(B)]
                if l >= L // 2:   # the skipped layers lie in the second half
                    on = [(S, g * (1 - skipped[b] / (L - L // 2)))
                          for b, (S, g) in enumerate(on)]
                f, w = _layer_cost(s, on, es)
                flops, nbytes = flops + f, nbytes + w
            if case["cache"]:
                nbytes += L * R * KV * d * 4 * 0.75
    elif kind == "decode":
        lens, groups, skipped = (_ints(case[k]) for k in ("cached", "groups", "skipped"))
        L = case["layers"]
        for l in range(L):
            on = [(1, g * (1 - (skipped[b] / (L - L // 2) if l >= L // 2 else 0.0)))
                  for b, g in enumerate(groups)]
            f, w = _layer_cost(s, on, es)
            kv = sum((n + 1) * g / GROUPS * KV * d * 4 for n, (_, g) in zip(lens, on))
            flops, nbytes = flops + f, nbytes + w + kv
        nbytes += len(lens) * D * 8
    elif kind == "train":
        S, B, L = case["n_vision"] + case["n_text"], case["batch"], case["layers"]
        w = (2 * A * d + 2 * KV * d + 3 * F) * D
        # forward, and the data gradients; attention: two products forward, five back
        flops = L * (2 * 2.0 * B * S * w + 3.5 * 2.0 * A * d * B * S * (S + 1))
        nbytes = L * w * es * 2 + B * S * D * (es * 2 + 8) + L * B * S * D * 8
    else:
        B, N, T = case["batch"], case["n_vision"], case["n_text"]
        L, P = case["layers"], case["prefix"]
        n1 = int(case["positive"] * N)
        for l in range(L):
            # after the prefix three of four groups; the projection to the budget cuts rows
            rows = n1 + T + 1 if l < P else min(n1 + T, int(case["budget"] * (N + T))) + 1
            f, w = _layer_cost(s, [(rows, GROUPS if l < P else 3)] * B, es)
            flops, nbytes = flops + f, nbytes + w
        nbytes += 2 * (PE_DIM * D + D * D) * es + B * (n1 + T + 1) * D * (es + 4)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # About four times the errors against exact().  float32 arithmetic: 6e-8 (gradients 1.1e-6) at the
    # tiny shape, up to 6.5e-6 in the gradients after sums of 11008 products;
    # 16-bit activations: 5e-4 (fp16) and 2.2e-3 (bf16) times the square root of
    # the layers, each of which rounds its activations a few times.
    if case["kind"] == "select":
        return "exact"
    if case["kind"] == "train" and case["shape"] != "tiny":
        return {"rel": 2.5e-5}
    if _dtype(case) == "f32":
        return {"rel": 1e-6 if case["kind"] == "prefill" else 5e-6}
    per_layer = 2e-3 if case["compute"] == "f16" else 1e-2
    return {"rel": per_layer * math.sqrt(case["layers"])}


# ------------------------------------------------------------------ 64-bit results
def _norm64(x, gain):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + EPS) * gain.double()


def _rope64(a, pos):
    """a [..., S, d] turned by the positions pos [S] (pairs r, r + d/2)."""
    d = a.shape[-1]
    w = THETA ** (-2.0 * torch.arange(d // 2, dtype=torch.float64, device=a.device) / d)
    phi = pos.double()[:, None] * w[None, :]
    c, sn = torch.cos(phi), torch.sin(phi)
    a1, a2 = a[..., :d // 2], a[..., d // 2:]
    return torch.cat([a1 * c - a2 * sn, a2 * c + a1 * sn], dim=-1)


def _attend64(q, k, v, first):
    """q [A, S, d], k and v [A, S', d]; query i sees keys 0 .. first + i."""
    sc = torch.matmul(q, k.transpose(1, 2).contiguous()) / math.sqrt(q.shape[-1])
    S, Sk = sc.shape[1], sc.shape[2]
    dead = torch.arange(Sk, device=q.device)[None, :] > first + torch.arange(S, device=q.device)[:, None]
    return torch.matmul(torch.softmax(sc.masked_fill(dead, -math.inf), dim=-1), v)


def _heads(y, n, d):
    return y.reshape(y.shape[0], n, d).transpose(0, 1).contiguous()


def _layer64(x, W, s, heads, chans, past=None, first=0, scale_o=None, scale_h=None):
    """One decoder layer in 64 bits on rows x [S][D]; heads, chans: the active
    ones (bool masks); past: cached (K, V) [KV][n][d] ahead of these rows.
    Returns the new rows and these rows' K and V."""
    A, KV, d = s["n_heads"], s["n_kv_heads"], s["head_dim"]
    S = x.shape[0]
    pos = torch.arange(first, first + S, device=x.device)
    u = _norm64(x, W["attn_norm"])
    q = _rope64(_heads(u @ W["wq"].double().t(), A, d), pos)
    k = _rope64(_heads(u @ W["wk"].double().t(), KV, d), pos)
    v = _heads(u @ W["wv"].double().t(), KV, d)
    ka, va = (k, v) if past is None else (torch.cat([past[0], k], 1), torch.cat([past[1], v], 1))
    rep = A // KV
    o = _attend64(q, ka.repeat_interleave(rep, 0), va.repeat_interleave(rep, 0), first)
    o = o * heads.double()[:, None, None] if scale_o is None else o * scale_o[:, None, None]
    x = x + o.transpose(0, 1).reshape(S, A * d) @ W["wo"].double().t()
    u = _norm64(x, W["ffn_norm"])
    g = u @ W["w_gate"].double().t()
    h = g * torch.sigmoid(g) * (u @ W["w_up"].double().t())
    h = h * (chans.double() if scale_h is None else scale_h)[None, :]
    return x + h @ W["w_down"].double().t(), k, v


def _select64(z, k):
    idx = torch.sort(z, descending=True, stable=True).indices[:k]
    return torch.sort(idx).values


def _kept_rows(kept, n):
    out = torch.full((n,), -1, dtype=torch.int32, device=kept.device)
    out[:kept.numel()] = kept.int()
    return out


def _masks64(hm, fm, F):
    heads = torch.from_numpy(np.ascontiguousarray(hm)).to("cuda").bool()
    chans = torch.from_numpy(np.ascontiguousarray(fm)).to("cuda").bool().repeat_interleave(F // GROUPS)
    return heads, chans


def exact(case, seed):
    with torch.no_grad():
        return _exact(case, seed)


def _exact(case, seed):
    st = prepare(case, seed)
    s = SHAPES[case["shape"]]
    kind = case["kind"]
    D, F, A, KV, d = (s[k] for k in ("d_model", "d_ffn", "n_heads", "n_kv_heads", "head_dim"))
    rep = A // KV
    if kind == "select" or kind == "prefill":
        B, N, T = len(st["keep"]), case["n_vision"], case["n_text"]
        kept = [_select64(st["scores"][b], int(st["keep"][b])) for b in range(B)]
        rows = [torch.cat([st["vision"][b][kept[b]], st["text"][b]]).double() for b in range(B)]
        idx = torch.stack([_kept_rows(k, N) for k in kept])
        if kind == "select":
            return {"kept": idx, "resid": torch.cat(rows)}
        lm, hm, fm = st["masks"]
        L = case["layers"]
        if case["cache"]:
            cache = torch.zeros((L, B, KV, 2, st["max_len"], d), dtype=torch.float64, device="cuda")
        for b in range(B):
            for l in range(L):
                if lm[b, l]:
                    heads, chans = _masks64(hm[b, l], fm[b, l], F)
                    rows[b], k, v = _layer64(rows[b], st["weights"][l], s, heads, chans)
                    if case["cache"]:
                        on = heads.reshape(KV, rep).any(1)
                        cache[l, b, on, 0, :k.shape[1]] = k[on]
                        cache[l, b, on, 1, :k.shape[1]] = v[on]
        out = {"kept": idx, "resid": torch.cat(rows)}
        if case["cache"]:
            out["cache"] = cache.reshape(-1)
        return out
    if kind == "decode":
        lm, hm, fm = st["masks"]
        L, B = case["layers"], len(st["lens"])
        cache = _cache_view(case, st["kv"]).double().reshape(L, B, KV, 2, st["max_len"], d)
        xs = []
        for b in range(B):
            x, n = st["emb"][b:b + 1].double(), int(st["lens"][b])
            for l in range(L):
                if not lm[b, l]:
                    continue
                heads, chans = _masks64(hm[b, l], fm[b, l], F)
                past = (cache[l, b, :, 0, :n], cache[l, b, :, 1, :n])
                x, k, v = _layer64(x, st["weights"][l], s, heads, chans, past, n)
                on = heads.reshape(KV, rep).any(1)
                cache[l, b, on, 0, n] = k[on, 0]
                cache[l, b, on, 1, n] = v[on, 0]
            xs.append(x)
        return {"x": torch.cat(xs), "cache": cache.reshape(-1)}
    if kind == "train":
        return _train64(case, st, s)
    return _controlled64(case, st, s)


def _train64(case, st, s):
    B, N, T, L, P = (case[k] for k in ("batch", "n_vision", "n_text", "layers", "prefix"))
    A, F = s["n_heads"], s["d_ffn"]
    zt, gt = st["z"] + st["zn"], st["g"] + st["gn"]
    y, yg = torch.sigmoid(zt.double() / TAU_TOK), torch.sigmoid(gt.double() / TAU_COMP)
    tm, um = zt > 0, gt > 0
    hidden, gz, gg = [], [], []
    all_heads = torch.ones(A, device="cuda")
    all_chans = torch.ones(F, device="cuda")
    for b in range(B):
        with torch.enable_grad():
            m = tm[b].double().requires_grad_(True)
            M = um[b].double().requires_grad_(True)
            x = torch.cat([st["vision"][b].double() * m[:, None], st["text"][b].double()])
            for l in range(L):
                u = M[(l - P) * GROUPS:(l - P + 1) * GROUPS] if l >= P else None
                so = None if u is None else u.repeat_interleave(A // GROUPS)
                sh = None if u is None else u.repeat_interleave(F // GROUPS)
                x, _, _ = _layer64(x, st["weights"][l], s, all_heads, all_chans, scale_o=so,
                                   scale_h=sh)
            wrt = [m, M] if M.numel() else [m]
            grads = torch.autograd.grad((x * st["grad"][b].double()).sum(), wrt)
        hidden.append(x.detach())
        gz.append(grads[0])
        gg.append(grads[1] if M.numel() else M.detach())
    return {"hidden": torch.stack(hidden), "token_mask": tm.to(torch.uint8),
            "unit_mask": um.to(torch.uint8),
            "grad_logits": torch.stack(gz) * y * (1 - y) / TAU_TOK,
            "grad_gate": torch.stack(gg) * yg * (1 - yg) / TAU_COMP}


def _encode64(x):
    w = PE_BASE ** (-2.0 * torch.arange(PE_DIM // 2, dtype=torch.float64, device="cuda") / PE_DIM)
    phi = float(x) * PE_SCALE * w
    return torch.stack([torch.sin(phi), torch.cos(phi)], dim=1).reshape(-1)


def _mlp64(t, name, x):
    h = t[name + "_w1"].double() @ x + t[name + "_b1"].double()
    h = 0.5 * h * (1.0 + torch.erf(h / math.sqrt(2.0)))
    return t[name + "_w2"].double() @ h + t[name + "_b2"].double()


def _cost(s, alphas, S):
    D, F = s["d_model"], s["d_ffn"]
    return sum(alphas) * ((8 * D * D + 6 * D * F) * S + 4 * D * S * S)


def _controlled64(case, st, s):
    B, N, T, L, P = (case[k] for k in ("batch", "n_vision", "n_text", "layers", "prefix"))
    A, F = s["n_heads"], s["d_ffn"]
    t = st["ctrl"].tensors
    budget = float(np.float32(case["budget"]))
    ones_h, ones_f = torch.ones(A, device="cuda"), torch.ones(F, device="cuda")
    e_b = _mlp64(t, "llm", _encode64(budget))
    out = dict(kept=[], resid=[], keep=[], layer_mask=[], head_mask=[], ffn_mask=[], gate_logits=[])
    for b in range(B):
        z = st["z"][b]
        count = int((z > 0).sum())
        kept = _select64(z, count)
        x = torch.cat([st["vision"][b][kept].double(), st["text"][b].double(), e_b[None, :]])
        for l in range(P):
            x, _, _ = _layer64(x, st["weights"][l], s, ones_h, ones_f)
        kap = torch.sigmoid(z.double()).mean()
        logits = t["gate_w"].double() @ (x[-1] + _mlp64(t, "kap", _encode64(kap))) + t["gate_b"].double()
        on = np.ones((L, GROUPS), np.uint8)
        on[P:] = (logits > 0).cpu().numpy().reshape(L - P, GROUPS)
        limit = budget * _cost(s, [1.0] * L, N + T)
        keep = count
        if budget < 1:
            # units leave, lowest logit first, only where the text alone does not fit
            conf = logits.cpu().numpy().reshape(L - P, GROUPS)
            order = sorted(((conf[l - P, j], -l, -j) for l in range(P, L) for j in range(GROUPS)
                            if on[l, j]))
            for _, l, j in order:
                if _cost(s, (on.sum(1) / GROUPS).tolist(), T) <= limit:
                    break
                on[-l, -j] = 0
            alphas = (on.sum(1) / GROUPS).tolist()
            keep = max((k for k in range(count + 1) if _cost(s, alphas, T + k) <= limit), default=0)
        final = _select64(z, keep)
        rows = torch.cat([torch.searchsorted(kept, final),
                          count + torch.arange(T + 1, device="cuda")])
        x = x[rows]
        for l in range(P, L):
            if on[l].any():
                heads, chans = _masks64(np.repeat(on[l], A // GROUPS), on[l], F)
                x, _, _ = _layer64(x, st["weights"][l], s, heads, chans)
        out["kept"].append(_kept_rows(final, N))
        out["resid"].append(x)
        out["keep"].append(keep)
        out["layer_mask"].append(on.any(1).astype(np.uint8))
        out["head_mask"].append(np.repeat(on, A // GROUPS, axis=1))
        out["ffn_mask"].append(on)
        out["gate_logits"].append(logits)
    return {"kept": torch.stack(out["kept"]), "resid": torch.cat(out["resid"]),
            "keep": np.array(out["keep"], np.int32), "layer_mask": np.stack(out["layer_mask"]),
            "head_mask": np.stack(out["head_mask"]), "ffn_mask": np.stack(out["ffn_mask"]),
            "gate_logits": torch.stack(out["gate_logits"])}
