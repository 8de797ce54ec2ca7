"""Each tile kind of the GEMMs, with every epilogue, at ragged sizes: one block run in full and then
refreshed on a quarter of its rows, against the same block in float64 torch.

The shapes are chosen so that between them the projections of the block take every kind of tile
(64 x 64, 128 x 128, 128 x 192, 192 x 192, 256 x 128, 256 x 256), with remainders of rows and columns,
Q / K / V boundaries inside a tile (hidden 64, 448, 1088) and the fewest stages along k (one).
"""
import math

import numpy as np
import pytest
import torch

from paper_2508_17588_amd import binding as B
from workloads import BLOCK_ADALN, get_config
from hero_testlib import assert_close, to_host_f64

pytestmark = pytest.mark.gpu


def weights(cfg, gen):
    d, f = cfg.hidden, cfg.ffn_dim

    def normal(*shape, std=0.02, mean=0.0):
        return (torch.randn(*shape, generator=gen, device="cuda") * std + mean).to(torch.bfloat16)

    w = {"w_qkv": normal(3 * d, d, std=0.04), "b_qkv": normal(3 * d), "w_o": normal(d, d), "b_o": normal(d),
         "w_ff1": normal(f, d), "b_ff1": normal(f), "w_ff2": normal(d, f), "b_ff2": normal(d),
         "ln1_g": normal(d, mean=1.0), "ln1_b": normal(d), "ln2_g": normal(d, mean=1.0), "ln2_b": normal(d)}
    if cfg.block_flags & BLOCK_ADALN:
        mod = torch.randn(12, d, generator=gen, device="cuda") * 0.1
        mod[2::3] += 1.0
        w["mod"] = mod.to(torch.bfloat16)
    return w


def norm(x, g, b, eps):
    return torch.nn.functional.layer_norm(x, (x.shape[1],), g, b, eps)


def block(cfg, w, x, rows, k_all, v_all):
    """K, V, the feature sum and the two branches of `rows`, which replace those rows of k_all / v_all first."""
    w = {n: t.double() for n, t in w.items()}
    d, hd = cfg.hidden, cfg.head_dim
    text = (rows < cfg.n_text)[:, None]

    def pick(i):                        # vector i of the six of a row's stream
        return torch.where(text, w["mod"][{0: 3, 1: 4, 2: 5, 6: 9, 7: 10, 8: 11}[i]], w["mod"][i])

    u = norm(x[rows], w["ln1_g"], w["ln1_b"], cfg.ln_eps)
    if "mod" in w:
        u = u * (1 + pick(1)) + pick(0)
    qkv = u @ w["w_qkv"].T + w["b_qkv"]
    k_all[rows], v_all[rows] = qkv[:, d:2 * d], qkv[:, 2 * d:]
    o = torch.empty_like(u)
    for h in range(cfg.n_heads):
        c = slice(h * hd, (h + 1) * hd)
        p = torch.softmax(qkv[:, c] @ k_all[:, c].T / math.sqrt(hd), dim=1)
        o[:, c] = p @ v_all[:, c]
    attn = o @ w["w_o"].T + w["b_o"]
    if "mod" in w:
        attn = attn * pick(2)
    u = norm(x[rows] + attn, w["ln2_g"], w["ln2_b"], cfg.ln_eps)
    if "mod" in w:
        u = u * (1 + pick(7)) + pick(6)
    h = torch.nn.functional.gelu(u @ w["w_ff1"].T + w["b_ff1"], approximate="tanh")
    ffn = h @ w["w_ff2"].T + w["b_ff2"]
    if "mod" in w:
        ffn = ffn * pick(8)
    return attn, attn + ffn


@pytest.mark.parametrize("heads,frames,height,width,n_text,flags,fp32", [
    (1, 1, 7, 7, 16, 0, True),               # hidden 64: one stage along k, Q, K and V inside one tile
    (7, 3, 9, 11, 3, BLOCK_ADALN, False),    # 300 rows
    (17, 3, 12, 19, 17, BLOCK_ADALN, True),  # 701 rows: 64 x 64 and 128 x 128
    (16, 4, 17, 19, 8, 0, False),            # 1300 rows: 128 x 192
    (17, 5, 17, 23, 77, BLOCK_ADALN, True),  # 2032 rows: 256 x 128, 128 x 128, 192 x 192
    (17, 4, 23, 27, 16, 0, False),           # 2500 rows: 192 x 192 and 256 x 256
])
def test_block_with_every_tile_kind(heads, frames, height, width, n_text, flags, fp32):
    d = heads * 64
    cfg = get_config("tiny", n_layers=1, n_shallow=1, hidden=d, n_heads=heads, head_dim=64, ffn_dim=4 * d, frames=frames,
                     height=height, width=width, n_text=n_text, block_flags=flags, resid_fp32=fp32)
    print(f"[case] {cfg.n_tokens} rows, hidden {d}, flags {flags}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    cache = B.HeroCache(B.make_config(cfg))
    w = weights(cfg, gen)
    cache.hero_set_layer_weights(0, w)
    n = cfg.n_tokens
    k_all = torch.zeros(n, d, dtype=torch.float64, device="cuda")
    v_all = torch.zeros_like(k_all)
    s_want, attn_want = torch.zeros_like(k_all), torch.zeros_like(k_all)
    idx = torch.zeros(n, dtype=torch.int32, device="cuda")
    for call in ("full", "refresh"):
        x = torch.randn(n, d, generator=gen, device="cuda").to(torch.float32 if fp32 else torch.bfloat16)
        x0 = x.double()
        if call == "full":
            rows = torch.arange(n, device="cuda")
            cache.hero_full_layer(0, x)
        else:
            n_sel = cache.hero_select(1, idx)
            rows = idx[:n_sel].long()
            cache.hero_refresh_layer(0, x, idx, n_sel)
        attn, s = block(cfg, w, x0, rows, k_all, v_all)
        s_want[rows], attn_want[rows] = s, attn
        torch.cuda.synchronize()
        assert_close(to_host_f64(cache.hero_cache_view(0, B.VIEW_K)), k_all.cpu().numpy(), f"{call} K")
        assert_close(to_host_f64(cache.hero_cache_view(0, B.VIEW_VT)[:, :n]), v_all.T.cpu().numpy(), f"{call} V^T")
        got_s = cache.hero_cache_view(0, B.VIEW_S_CUR)
        assert_close(to_host_f64(got_s), s_want.cpu().numpy(), f"{call} S", stored_parts=[attn_want.cpu().numpy()])
        # the residual add takes the features as stored: one fp32 addition, then the stream's own rounding
        add = x0 + got_s.double()
        err = (x.double() - add).abs()
        bound = (2.0 ** -23 if fp32 else 2.0 ** -8) * add.abs() + 1e-7
        assert bool((err <= bound).all()), f"{call} x: off by {float((err - bound).max())}"
    cache.close()


@pytest.mark.parametrize("m,n,k", [(1, 64, 64), (65, 192, 320), (326, 256, 1024), (691, 3072, 1024), (1755, 3072, 3072),
                                   (2925, 3072, 1024), (2032, 4160, 1024), (1987, 1984, 1088)])
def test_linear_tile_edges(m, n, k):
    print(f"[case] linear {m} x {n} x {k}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m)
    a = torch.randn(m, k, generator=gen, device="cuda").to(torch.bfloat16)
    w = (torch.randn(n, k, generator=gen, device="cuda") * 0.02).to(torch.bfloat16)
    bias = torch.randn(n, generator=gen, device="cuda").to(torch.bfloat16)
    guard = torch.full((m + 1, n), 7.0, dtype=torch.bfloat16, device="cuda")     # the row past the end stays as it is
    want = a.double() @ w.double().T + bias.double()
    for act in (0, 1):
        guard.fill_(7.0)
        B.hero_linear(a, w, bias, guard, act)
        ref = torch.nn.functional.gelu(want, approximate="tanh") if act else want
        torch.cuda.synchronize()
        assert bool((guard[m] == 7.0).all())
        assert_close(to_host_f64(guard[:m]), ref.cpu().numpy(), f"linear {m}x{n}x{k} act {act}")
