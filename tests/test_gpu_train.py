"""GPU parity of the training-time masked decoder (svl_train_step) against
oracle/training.py's masked_train_step, through the C ABI.

Per sample: token and unit masks exact (the decisions compare float32
z + xi with 0 on both sides, and rounding keeps the sign of a sum); the final
hidden states within 1e-4 normwise relative error (the float32 bar); the
gate-logit gradients within TOL_GRAD normwise; each token-logit gradient
within TOL_GRAD of its condition scale: dL/dz_i is the dot product
(dL/dX_0[i] . v_i) y_i (1 - y_i) / tau, whose rounding error is bounded by
the error of dL/dX_0 times sum_d |dL/dX_0[i][d] v_i[d]| y_i (1 - y_i) / tau,
so that scale (from the oracle) divides the difference.  (Gradients of
dropped tokens pass through the RMSNorm of a zero row, which scales them by
eps^(-1/2): they differ from the kept tokens' by orders, and a normwise
measure over all tokens would see only them.)

"""
import dataclasses

import numpy as np
import pytest
import torch

import paper_2607_20357_amd as svl
import workloads as W
from gpu_helpers import host_layer
from oracle import training as ot

pytestmark = pytest.mark.gpu

TOL_HIDDEN = 1e-4
TOL_GRAD = 1e-3


def _normwise(got, want):
    got = np.asarray(got, np.float64)
    want = np.asarray(want, np.float64)
    if want.size == 0:
        return 0.0
    den = np.abs(want).max()
    return float(np.abs(got - want).max() / den) if den > 0 else float(np.abs(got).max())


def _run(w, seed, prefix, units, tau_tok=0.7, tau_comp=1.3, drop_first=False, noise=True):
    s = w.shape
    B, N, T, D, L = w.batch, w.n_vision, w.n_text, s.d_model, s.n_layers
    S = N + T
    print(f"train {w.name} B={B} N={N} T={T} L={L} P={prefix} U={units} seed={seed}", flush=True)
    cfg = svl.make_config(s)
    vision, text = W.draw_hidden(w, seed, device="cuda")
    layers = [W.draw_layer_weights(w, l, seed, device="cuda") for l in range(L)]
    rng = np.random.default_rng(seed + 101)
    nl = (L - prefix) * units
    z = rng.normal(0.3, 1.5, (B, N)).astype(np.float32)
    if N:
        z[:, 0] = -20.0 if drop_first else 20.0
    g = rng.normal(0.6, 1.5, (B, nl)).astype(np.float32)
    xi = rng.logistic(0, 1, (B, N)).astype(np.float32) if noise else None
    xg = rng.logistic(0, 1, (B, nl)).astype(np.float32) if noise else None
    G = rng.standard_normal((B, S, D)).astype(np.float32)
    t = lambda a: None if a is None else torch.from_numpy(a).cuda()
    prm = svl.svl_train_params(tau_tok, tau_comp, prefix, units)
    ws = svl.alloc_train_workspace(cfg, prm, B, N, T)
    out = svl.svl_train_step(cfg, svl.LayerTable(layers), prm, t(z), t(g), vision, text, t(G), ws,
                             token_noise=t(xi), gate_noise=t(xg))
    torch.cuda.synchronize()
    got = {k: v.cpu().numpy() for k, v in out.items()}

    hl = [host_layer(l) for l in layers]
    vis, txt = W.as_f32(vision), W.as_f32(text)
    errs = {"hidden": 0.0, "token": 0.0, "gate": 0.0}
    for b in range(B):
        ref = ot.masked_train_step(s, lambda l: hl[l], vis[b], txt[b], z[b].astype(np.float64),
                                   g[b].astype(np.float64), G[b], prefix, units, tau_tok, tau_comp,
                                   xi_tok=None if xi is None else xi[b].astype(np.float64),
                                   xi_gate=None if xg is None else xg[b].astype(np.float64))
        np.testing.assert_array_equal(got["token_mask"][b], ref.token_mask)
        np.testing.assert_array_equal(got["unit_mask"][b], ref.unit_mask)
        errs["hidden"] = max(errs["hidden"], _normwise(got["hidden"][b], ref.hidden))
        v = z[b].astype(np.float64) + (0.0 if xi is None else xi[b].astype(np.float64))
        y = 1.0 / (1.0 + np.exp(-v / tau_tok))
        cond = np.sum(np.abs(ref.grad_x0[:N] * vis[b]), axis=1) * y * (1.0 - y) / tau_tok
        diff = np.abs(got["grad_logits"][b].astype(np.float64) - ref.grad_z)
        errs["token"] = max(errs["token"], float(np.max(diff / cond, initial=0.0)))
        errs["gate"] = max(errs["gate"], _normwise(got["grad_gate"][b], ref.grad_gate))
    print("  " + ", ".join(f"{k} {v:.2e}" for k, v in errs.items()), flush=True)
    assert errs["hidden"] <= TOL_HIDDEN, errs
    for k in ("token", "gate"):
        assert errs[k] <= TOL_GRAD, (k, errs)
    return got


def _tiny(batch=2):
    return W.scaled(W.get_workload("tiny_f32"), batch=batch, name="tiny_f32_train")


@pytest.mark.parametrize("prefix,units", [(0, 4), (1, 4), (1, 1), (2, 1)])
def test_train_tiny_f32(prefix, units):
    _run(_tiny(), 3, prefix, units)


def test_train_tiny_first_token_dropped_and_no_noise():
    _run(_tiny(), 4, 1, 4, drop_first=True, noise=False)


def test_train_forward_only_matches_the_full_step():
    """Without grad_hidden the call runs the forward alone: same hidden states
    and masks, and no gradient outputs."""
    w = _tiny()
    s = w.shape
    cfg = svl.make_config(s)
    vision, text = W.draw_hidden(w, 5, device="cuda")
    layers = svl.LayerTable([W.draw_layer_weights(w, l, 5, device="cuda") for l in range(2)])
    rng = np.random.default_rng(5)
    z = torch.from_numpy(rng.normal(0, 2, (2, w.n_vision)).astype(np.float32)).cuda()
    g = torch.from_numpy(rng.normal(0, 2, (2, 8)).astype(np.float32)).cuda()
    G = torch.from_numpy(rng.standard_normal((2, w.n_vision + w.n_text, s.d_model))
                         .astype(np.float32)).cuda()
    prm = svl.svl_train_params(0.5, 0.5, 0, 4)
    ws = svl.alloc_train_workspace(cfg, prm, 2, w.n_vision, w.n_text)
    a = svl.svl_train_step(cfg, layers, prm, z, g, vision, text, None, ws)
    b = svl.svl_train_step(cfg, layers, prm, z, g, vision, text, G, ws)
    torch.cuda.synchronize()
    assert "grad_logits" not in a
    assert torch.equal(a["hidden"], b["hidden"])
    assert torch.equal(a["token_mask"], b["token_mask"]) and torch.equal(a["unit_mask"], b["unit_mask"])


@pytest.mark.parametrize("units", [4, 1])
def test_train_scaled_7b_bf16(units):
    w = W.scaled(W.get_workload("llava7b_b1_keep25"), n_layers=3, d_model=512, n_heads=4,
                 n_kv_heads=4, d_ffn=1024, batch=2, n_vision=144, n_text=32,
                 name="llava7b_train_scaled")
    _run(w, 6, 1, units)


def test_train_scaled_gqa_bf16():
    w = W.scaled(W.get_workload("gqa7b_hires_b2"), n_layers=2, d_model=512, n_heads=4,
                 n_kv_heads=2, d_ffn=1024, batch=2, n_vision=160, n_text=48,
                 name="gqa7b_train_scaled")
    _run(w, 7, 0, 4)


def test_train_head_dim_32_gqa():
    """32-dimensional heads (8 query heads over 4 K/V heads, two per group)
    and 130 rows, three 64-row tiles with a ragged last one."""
    base = _tiny()
    shape = dataclasses.replace(base.shape, n_heads=8, n_kv_heads=4, head_dim=32)
    w = dataclasses.replace(base, shape=shape, n_vision=100, n_text=30, name="tiny_hd32_train")
    _run(w, 9, 1, 4)


@pytest.mark.parametrize("n_vision,n_text,prefix", [(0, 40, 1), (60, 0, 1), (40, 24, 2)])
def test_train_edge_shapes(n_vision, n_text, prefix):
    """No vision tokens (no token logits or gradients), no text tokens, and a
    prefix covering every layer (no gate logits or gradients)."""
    w = dataclasses.replace(_tiny(), n_vision=n_vision, n_text=n_text,
                            name=f"tiny_train_n{n_vision}_t{n_text}_p{prefix}")
    got = _run(w, 10, prefix, 4)
    assert got["token_mask"].shape == (2, n_vision)
    assert got["unit_mask"].shape == (2, (w.shape.n_layers - prefix) * 4)


def test_train_headline_width():
    """The headline's width (d_model 4096, 32 heads x 128, FFN 11008; 576 vision
    and 64 text tokens), two layers, the layer-head controller from layer 1."""
    w = W.scaled(W.get_workload("llava7b_b1_keep25"), n_layers=2, name="llava7b_train_width")
    _run(w, 8, 1, 4)


@pytest.mark.parametrize("batch,n_vision,n_text", [(1, 1, 0), (1, 60, 4), (1, 100, 27), (2, 50, 14),
                                                   (1, 120, 9), (3, 77, 9)])
def test_train_bf16_product_tile_edges(batch, n_vision, n_text):
    """bf16-weight products (128 x 256 output tiles, K in steps of 32, K pieces):
    1, 64, 127, 128, 129 and 258 rows; 320 output columns (a full tile and a
    ragged one), 64 columns (K / V heads) and 192 + 64 + 64 columns side by side,
    reductions of 192 and 64 beside each other along K, and samples that cross
    a tile's rows under their own unit masks.  Without noise: with it the first
    token's 1 - y falls below float64's resolution in the oracle."""
    base = _tiny(batch)
    shape = dataclasses.replace(base.shape, d_model=320, n_heads=3, n_kv_heads=1, head_dim=64,
                                d_ffn=768, n_groups=3, dtype="bf16")
    w = dataclasses.replace(base, shape=shape, n_vision=n_vision, n_text=n_text,
                            name=f"train_edges_b{batch}_{n_vision}_{n_text}")
    _run(w, 12, 1, 3, noise=False)


def test_train_without_room_for_every_layers_set():
    """A workspace of svl_train_workspace_bytes holds one layer's forward set:
    each forward runs again before its backward, with the same results."""
    w = W.scaled(W.get_workload("llava7b_b1_keep25"), n_layers=3, d_model=512, n_heads=4,
                 n_kv_heads=4, d_ffn=1024, batch=2, n_vision=70, n_text=20, name="train_small_ws")
    s = w.shape
    B, N, T, D = 2, 70, 20, s.d_model
    cfg = svl.make_config(s)
    vision, text = W.draw_hidden(w, 13, device="cuda")
    layers = svl.LayerTable([W.draw_layer_weights(w, l, 13, device="cuda") for l in range(3)])
    rng = np.random.default_rng(13)
    t = lambda *shape: torch.from_numpy(rng.standard_normal(shape).astype(np.float32)).cuda()
    z, g, G = t(B, N), t(B, 8), t(B, N + T, D)
    prm = svl.svl_train_params(0.5, 0.5, 1, 4)
    ws = svl.alloc_train_workspace(cfg, prm, B, N, T)
    a = svl.svl_train_step(cfg, layers, prm, z, g, vision, text, G, ws)
    small = svl.svl_train_workspace_bytes(cfg, prm, B, N, T)
    assert small < ws.numel()
    b = svl.svl_train_step(cfg, layers, prm, z, g, vision, text, G, ws[:small])
    torch.cuda.synchronize()
    for k in a:
        assert torch.equal(a[k], b[k]), k


@pytest.mark.parametrize("batch,n_vision,n_text,d_model,d_ffn", [
    (1, 1, 0, 256, 688), (1, 20, 13, 144, 272), (2, 40, 25, 528, 1040), (1, 600, 41, 1024, 1088)])
def test_train_f32_product_tiles(batch, n_vision, n_text, d_model, d_ffn):
    """Float32-weight products on both sides of the 32 x 32 / 64 x 64 tile rule: 1,
    33, 130 and 641 rows; widths and reductions that end a 64-column step after
    16 and 32 columns; a reduction just above the rule's 1024."""
    base = _tiny(batch)
    shape = dataclasses.replace(base.shape, d_model=d_model, d_ffn=d_ffn)
    w = dataclasses.replace(base, shape=shape, n_vision=n_vision, n_text=n_text,
                            name=f"train_f32_b{batch}_{n_vision}_{n_text}_{d_model}")
    _run(w, 14, 1, 4, noise=False)


@pytest.mark.parametrize("d_model,heads,kv,head_dim,d_ffn,batch,n_vision,n_text", [
    (320, 3, 1, 64, 768, 1, 100, 27), (1024, 8, 2, 128, 2816, 2, 40, 9),
    (4096, 32, 32, 128, 11008, 1, 90, 10), (3584, 28, 4, 128, 18944, 1, 1, 0)])
def test_train_required_workspace_same_bits(d_model, heads, kv, head_dim, d_ffn, batch, n_vision, n_text):
    """The slices of a bf16 product's K pieces lie in regions that are dead at
    its launch.  A step in the required bytes, which runs each forward again
    before its backward, gives the bits of one that keeps every layer's set,
    whatever the workspace held before."""
    base = _tiny(batch)
    units = 1 if heads == 3 else 4
    shape = dataclasses.replace(base.shape, n_layers=2, d_model=d_model, n_heads=heads, n_kv_heads=kv,
                                head_dim=head_dim, d_ffn=d_ffn, n_groups=units, dtype="bf16")
    w = dataclasses.replace(base, shape=shape, n_vision=n_vision, n_text=n_text, name="train_slices")
    print(f"train workspace {d_model} {heads}/{kv}x{head_dim} {d_ffn} {batch}x({n_vision}+{n_text})",
          flush=True)
    cfg = svl.make_config(shape)
    vision, text = W.draw_hidden(w, 15, device="cuda")
    layers = svl.LayerTable([W.draw_layer_weights(w, l, 15, device="cuda") for l in range(2)])
    rng = np.random.default_rng(15)
    t = lambda *sh: torch.from_numpy(rng.standard_normal(sh).astype(np.float32)).cuda()
    z, g, G = t(batch, n_vision), t(batch, units), t(batch, n_vision + n_text, d_model)
    prm = svl.svl_train_params(0.5, 0.5, 1, units)
    full = svl.alloc_train_workspace(cfg, prm, batch, n_vision, n_text)
    small = svl.svl_train_workspace_bytes(cfg, prm, batch, n_vision, n_text)
    assert small < full.numel()
    outs = []
    for ws, fill in ((full, 0), (full, 255), (full[:small], 255)):
        ws.fill_(fill)
        outs.append(svl.svl_train_step(cfg, layers, prm, z, g, vision, text, G, ws))
    torch.cuda.synchronize()
    for o in outs[1:]:
        for k in o:
            assert torch.equal(o[k], outs[0][k]), k


@pytest.mark.parametrize("name", ["w_down", "w_up", "text"])
def test_train_bf16_infinite_weight(name):
    """One infinite bf16 weight: its output column is +inf or -inf by the sign
    of the row's factor, as a float32 product gives it (a factor's zero low
    term, one in about 256, times infinity would be NaN); and an infinite
    column of the activations makes every output infinite.  A NaN input alone
    ("text") makes its row and the later rows of its sample NaN."""
    base = _tiny(2)
    shape = dataclasses.replace(base.shape, n_layers=1, d_model=320, n_heads=4, n_kv_heads=2, head_dim=64,
                                d_ffn=768, n_groups=4, dtype="bf16")
    w = dataclasses.replace(base, shape=shape, n_vision=0, n_text=700, name="train_inf_weight")
    cfg = svl.make_config(shape)
    vision, text = W.draw_hidden(w, 16, device="cuda")
    layer = dict(W.draw_layer_weights(w, 0, 16, device="cuda"))
    if name == "text":
        text[1, 400, 7] = float("nan")
    else:
        layer[name] = layer[name].clone()
        layer[name][300, 129] = float("inf")    # [out][in]
    prm = svl.svl_train_params(0.5, 0.5, 1, 4)
    ws = svl.alloc_train_workspace(cfg, prm, 2, 0, 700)
    z, g = torch.zeros(2, 0, device="cuda"), torch.zeros(2, 0, device="cuda")
    out = svl.svl_train_step(cfg, svl.LayerTable([layer]), prm, z, g, vision, text, None, ws)
    torch.cuda.synchronize()
    hidden = out["hidden"].cpu().numpy()
    hl = host_layer(layer)
    for b in range(2):
        with np.errstate(all="ignore"):
            ref, _ = ot.masked_forward(shape, lambda l: hl, W.as_f32(vision)[b], W.as_f32(text)[b],
                                       np.zeros(0), np.zeros((0, 4)), 1, 4)
        if name == "w_down":
            assert np.isinf(ref[:, 300]).all()
            np.testing.assert_array_equal(hidden[b][:, 300], ref[:, 300])
            cols = np.arange(320) != 300
            assert _normwise(hidden[b][:, cols], ref[:, cols]) <= TOL_HIDDEN
        elif name == "text":
            # (the oracle's masked probabilities, 0 times NaN, reach earlier rows too)
            assert np.isfinite(hidden[b][:384]).all()
            assert np.isnan(hidden[b][400:]).all() if b else np.isfinite(hidden[b]).all()
        else:
            assert np.isinf(ref).all()
            np.testing.assert_array_equal(hidden[b], ref)


def _truncated(x, bits):
    """x as float32 with its significand cut to `bits` (8 per bf16 term)."""
    v = x.to(torch.float32).contiguous().view(torch.int32)
    return (v & ~((1 << (24 - bits)) - 1)).view(torch.float32).double()


def _forward64(s, layers, x, masks, prefix, units, bits=None):
    """The masked decoder's forward of one sample in float64 (CPU); with `bits`,
    every product's activations are cut to that many significand bits."""
    cut = (lambda t: t) if bits is None else (lambda t: _truncated(t, bits))
    A, KV, d, S = s.n_heads, s.n_kv_heads, s.head_dim, x.shape[0]
    w = s.rope_theta ** (-2.0 * torch.arange(d // 2, dtype=torch.float64) / d)
    phi = torch.arange(S, dtype=torch.float64)[:, None] * w[None, :]

    def rope(a):
        a1, a2 = a[..., :d // 2], a[..., d // 2:]
        c, sn = torch.cos(phi)[:, None], torch.sin(phi)[:, None]
        return torch.cat([a1 * c - a2 * sn, a2 * c + a1 * sn], dim=-1)

    def norm(t, g):
        return t * torch.rsqrt((t * t).mean(-1, keepdim=True) + s.rms_eps) * g
    for l, W_ in enumerate(layers):
        m = torch.ones(units, dtype=torch.float64) if l < prefix else masks[l - prefix]
        u = cut(norm(x, W_["attn_norm"]))
        q = rope((u @ W_["wq"].t()).reshape(S, A, d))
        k = rope((u @ W_["wk"].t()).reshape(S, KV, d)).repeat_interleave(A // KV, 1)
        v = (u @ W_["wv"].t()).reshape(S, KV, d).repeat_interleave(A // KV, 1)
        sc = torch.matmul(q.transpose(0, 1), k.permute(1, 2, 0)) / d ** 0.5
        sc = sc.masked_fill(torch.ones(S, S).triu(1).bool(), -float("inf"))
        o = torch.matmul(torch.softmax(sc, -1), v.transpose(0, 1).contiguous()).transpose(0, 1)
        o = (o * m.repeat_interleave(A // units)[None, :, None]).reshape(S, A * d)
        x = x + cut(o) @ W_["wo"].t()
        u = cut(norm(x, W_["ffn_norm"]))
        g = u @ W_["w_gate"].t()
        h = g * torch.sigmoid(g) * (u @ W_["w_up"].t()) * m.repeat_interleave(s.d_ffn // units)[None, :]
        x = x + cut(h) @ W_["w_down"].t()
    return x


@pytest.mark.parametrize("batch,rows", [(1, 1), (1, 64), (1, 129), (3, 86)])
def test_train_bf16_products_keep_all_three_terms(batch, rows):
    """bf16-weight products at tile edges, close enough to see the third term.
    Hidden states: float32 sums of up to 768 products in runs of 512, and the
    float32 norms, softmax and residuals of two layers, about 10 roundings of
    2^-24 in a row of size one: 6e-7 normwise.  With 16 bits of each factor the
    products alone are off by 2^-17 of their size, the same way for every
    factor."""
    base = _tiny(batch)
    shape = dataclasses.replace(base.shape, d_model=320, n_heads=3, n_kv_heads=1, head_dim=64,
                                d_ffn=768, n_groups=3, dtype="bf16")
    w = dataclasses.replace(base, shape=shape, n_vision=0, n_text=rows, name="train_terms")
    cfg = svl.make_config(shape)
    vision, text = W.draw_hidden(w, 17, device="cuda")
    layers = [W.draw_layer_weights(w, l, 17, device="cuda") for l in range(2)]
    rng = np.random.default_rng(17)
    g = torch.from_numpy(rng.normal(0.6, 1.5, (batch, 3)).astype(np.float32)).cuda()
    prm = svl.svl_train_params(0.7, 1.3, 1, 3)
    ws = svl.alloc_train_workspace(cfg, prm, batch, 0, rows)
    out = svl.svl_train_step(cfg, svl.LayerTable(layers), prm, torch.zeros(batch, 0, device="cuda"), g,
                             vision, text, None, ws)
    hidden = out["hidden"].double().cpu()
    hl = [{k: v.double().cpu() for k, v in l.items()} for l in layers]
    for b in range(batch):
        masks = (g[b].cpu() > 0).double().reshape(1, 3)
        x = text[b].double().cpu()
        ref = _forward64(shape, hl, x, masks, 1, 3)
        den = ref.abs().max()
        err = float((hidden[b] - ref).abs().max() / den)
        two = float((_forward64(shape, hl, x, masks, 1, 3, bits=16) - ref).abs().max() / den)
        print(f"train terms batch {batch} rows {rows}: {err:.2e}, two terms {two:.2e}", flush=True)
        assert err <= 6e-7
        assert two > 1.2e-6


def test_train_bf16_negative_zeros():
    """-0 among the factors of bf16-weight products, whose three-term split has no
    place for it: zeroed tokens under gains of both signs, unit masks of 0 times
    negative values, text rows of -0 and a gradient with entries of -0.  Same
    bits as with +0 in the caller's tensors, and the float64 forward's values."""
    base = _tiny(2)
    shape = dataclasses.replace(base.shape, n_layers=2, d_model=320, n_heads=4, n_kv_heads=2, head_dim=64,
                                d_ffn=768, n_groups=4, dtype="bf16")
    N, T = 60, 30
    w = dataclasses.replace(base, shape=shape, n_vision=N, n_text=T, name="train_neg_zero")
    cfg = svl.make_config(shape)
    vision, text = W.draw_hidden(w, 18, device="cuda")
    layers = [dict(W.draw_layer_weights(w, l, 18, device="cuda")) for l in range(2)]
    for l in layers:
        for name in ("attn_norm", "ffn_norm"):
            l[name] = l[name].clone()
            l[name][::2] *= -1
    rng = np.random.default_rng(18)
    t = lambda *sh: torch.from_numpy(rng.standard_normal(sh).astype(np.float32)).cuda()
    z, G = t(2, N), t(2, N + T, 320)
    g = torch.tensor([[1.0, -1.0, 1.0, -1.0], [-1.0, 1.0, -1.0, -1.0]], device="cuda")
    G[:, ::3] = 0.0
    text[:, 5:9] = 0.0
    prm = svl.svl_train_params(0.7, 1.3, 1, 4)
    ws = svl.alloc_train_workspace(cfg, prm, 2, N, T)
    table = svl.LayerTable(layers)
    outs = []
    for zero in (0.0, -0.0):
        G[:, ::3] = zero
        text[:, 5:9] = zero
        ws.fill_(255)
        outs.append(svl.svl_train_step(cfg, table, prm, z, g, vision, text, G, ws))
    torch.cuda.synchronize()
    for k, v in outs[0].items():
        assert torch.equal(v, outs[1][k]), k
        assert torch.isfinite(v.float()).all(), k
    hl = [{k: v.double().cpu() for k, v in l.items()} for l in layers]
    for b in range(2):
        x = torch.cat([vision[b].double() * (z[b] > 0).double()[:, None], text[b].double()]).cpu()
        ref = _forward64(shape, hl, x, (g[b].cpu() > 0).double().reshape(1, 4), 1, 4)
        err = float((outs[1]["hidden"][b].double().cpu() - ref).abs().max() / ref.abs().max())
        assert err <= 1e-6, err
