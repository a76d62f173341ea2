"""The bf16 mode's QKV and gate/up products take the normed rows as two bf16
terms.  One layer's parity bar (2e-2) cannot see the second term, so these tests
look where nothing else rounds: the cached K and V rows, and the SwiGLU output
read through a down projection that picks single channels.

Tolerance, per value v of a row set with root mean square s: one rounding to
bf16 (8 significant bits: 2^-8 |v|), and the rest of the two-term row, at
most 2^-17 of each factor, with the float32 sums: under 1e-4 s (for sums of K
products of random signs it grows as the row's own value does, so it stays
near 2^-17 s = 8e-6 s; 1e-4 s leaves room for the largest of 10^6 values).
Rows of one term miss it: their error is near 1e-3 s whatever v is."""
import dataclasses

import numpy as np
import pytest
import torch

import paper_2607_20357_amd as svl
import workloads as W

pytestmark = pytest.mark.gpu

D = 832          # 13 K chunks: three weight stages and one chunk
# row blocks per tile: 1 of one wave; 2; 5; 9; 12; 13; 16
ROWS = [9, 17, 70, 144, 190, 208, 250]


def _bf16(x):
    return x.float().to(torch.bfloat16).double()


def _normed(x, gain, eps):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + eps) * gain.double()


def _misses(got, want):
    """Largest excess over the tolerance, in units of the root mean square."""
    s = float(want.pow(2).mean().sqrt())
    return float(((got - want).abs() - 2.0 ** -8 * want.abs()).max()) / s


def _rope(a, theta):
    """a [S][heads][d], row i at position i."""
    d = a.shape[-1]
    w = theta ** (-2.0 * torch.arange(d // 2, dtype=torch.float64, device=a.device) / d)
    phi = torch.arange(a.shape[0], dtype=torch.float64, device=a.device)[:, None] * w[None, :]
    c, s = torch.cos(phi)[:, None, :], torch.sin(phi)[:, None, :]
    a1, a2 = a[..., :d // 2], a[..., d // 2:]
    return torch.cat([a1 * c - a2 * s, a2 * c + a1 * s], dim=-1)


# 24 blocks a head: launches of 264 .. 2040 blocks, tiles of 2, 3, 4, 5, 6 and 8
@pytest.mark.parametrize("heads", [11, 24, 32, 48, 60, 85])
def test_two_term_kv_rows(heads):
    base = W.get_workload("tiny_f32").shape
    shape = dataclasses.replace(base, n_layers=1, d_model=D, n_heads=heads, n_kv_heads=heads,
                                head_dim=128, d_ffn=64, n_groups=1, dtype="bf16")
    cfg = svl.make_config(shape, compute="bf16")
    dev = "cuda"
    w = W.Workload(name="two_term", shape=shape, batch=1, n_vision=0, n_text=0)
    weights = W.draw_layer_weights(w, 0, 21, device=dev)
    for rows in ROWS:
        print(f"two-term K/V, {heads} heads, {rows} rows", flush=True)
        g = torch.Generator(device=dev).manual_seed(rows)
        text = torch.randn(1, rows, D, generator=g, device=dev).to(torch.bfloat16)
        vision = torch.zeros(1, 0, D, dtype=torch.bfloat16, device=dev)
        scores = torch.zeros(1, 0, device=dev)
        kept = torch.zeros(1, 0, dtype=torch.int32, device=dev)
        resid = torch.empty(rows, D, device=dev)
        kv = svl.alloc_kv_cache(cfg, 1, rows, dev)
        ws = svl.alloc_workspace(cfg, 1, rows, dev).fill_(255)
        svl.svl_prefill_cache(cfg, [weights], np.zeros(1, np.int32), scores, vision, text,
                              np.ones((1, 1), np.uint8), np.ones((1, 1, heads), np.uint8),
                              np.zeros((1, 1, 1), np.uint8), kept, resid, kv, rows, ws)
        got = kv.view(torch.bfloat16).double().reshape(heads, 2, rows, 128)
        xn = _normed(text[0].double(), weights["attn_norm"], shape.rms_eps)

        def cached(rows_in):
            k = _rope((rows_in @ weights["wk"].double().t()).reshape(rows, heads, 128), shape.rope_theta)
            v = (rows_in @ weights["wv"].double().t()).reshape(rows, heads, 128)
            return torch.stack([k, v]).permute(2, 0, 1, 3)
        want = cached(xn)
        assert _misses(got, want) <= 1e-4
        assert _misses(_bf16(cached(_bf16(xn))), want) > 3e-4     # one term would fail


@pytest.mark.parametrize("blocks", [1, 2, 3, 4, 5, 6, 8])
def test_two_term_swiglu_rows(blocks):
    """Gate/up tiles of every block count (d_ffn fills 256 tiles of that width)."""
    base = W.get_workload("tiny_f32").shape
    F = 2048 * blocks
    shape = dataclasses.replace(base, n_layers=1, d_model=D, n_heads=13, n_kv_heads=13, head_dim=64,
                                d_ffn=F, n_groups=1, dtype="bf16")
    cfg = svl.make_config(shape, compute="bf16")
    dev = "cuda"
    w = W.Workload(name="two_term", shape=shape, batch=1, n_vision=0, n_text=0)
    weights = dict(W.draw_layer_weights(w, 0, 22, device=dev))
    for name in ("w_gate", "w_up"):     # gate and up values of about one
        weights[name] = (weights[name].float() / weights[name].float().std() / D ** 0.5).to(torch.bfloat16)
    for rows in ROWS:
        print(f"two-term gate/up, {blocks} blocks, {rows} rows", flush=True)
        g = torch.Generator(device=dev).manual_seed(100 + rows)
        pick = torch.randperm(F, generator=g, device=dev)[:D]     # output i is channel pick[i]
        down = torch.zeros(D, F, device=dev)
        down[torch.arange(D, device=dev), pick] = 1.0
        weights["w_down"] = down.to(torch.bfloat16)
        x = torch.randn(rows, D, generator=g, device=dev) * 2.0 ** -6
        resid = x.clone()
        ws = svl.alloc_workspace(cfg, 1, rows, dev).fill_(255)
        svl.svl_layer_forward(cfg, 0, weights, np.array([0, rows], np.int32), np.ones(1, np.uint8),
                              np.zeros((1, 13), np.uint8), np.ones((1, 1), np.uint8), resid, ws)
        got = resid.double() - x.double()
        xn = _normed(x.double(), weights["ffn_norm"], shape.rms_eps)

        def hidden(rows_in):
            gt = rows_in @ weights["w_gate"].double().t()
            return (gt * torch.sigmoid(gt) * (rows_in @ weights["w_up"].double().t()))[:, pick]
        want = hidden(xn)
        assert _misses(got, want) <= 1e-4
        assert _misses(_bf16(hidden(_bf16(xn))), want) > 3e-4     # one term would fail
