"""One block in plain float64 torch, a layer of the library run against it, and the shapes it is run at."""
import math

import torch

from paper_2508_17588_amd import binding as B
from workloads import BLOCK_ADALN, get_config
from hero_testlib import assert_close, to_host_f64


# Blocks between which each of a layer's four GEMMs, on all rows and on listed ones, takes every kind of tile, with remainders of
# rows and columns and Q / K / V boundaries inside tiles (tests/test_routes.py holds them to it, together with the shapes of
# the narrow models and of the cut tiles).  Heads of 64 channels, FFN width, frames, height, width, text rows, ratio,
# patch height and width.
BLOCKS = [
    (1, 320, 1, 11, 7, 8, 0.5, 3, 5),            # 85 and 40 rows, one stage along k
    (5, 320, 1, 7, 9, 3, 0.1, 2, 3),             # 66 and 12 rows
    (13, 1024, 6, 10, 26, 3, 0.75, 2, 3),        # 1563 and 1290
    (1, 9216, 3, 13, 20, 3, 0.75, 2, 2),         # 783 and 600
    (1, 9216, 4, 18, 13, 77, 0.75, 3, 5),        # 1013 and 696
    (5, 6144, 2, 35, 18, 3, 0.75, 2, 3),         # 1263 and 1044
    (17, 1024, 6, 27, 28, 17, 0.75, 2, 3),       # 4553 and 3780
    (32, 4096, 3, 33, 45, 17, 0.75, 2, 3),       # 4472 and 3690
    (28, 64, 5, 15, 43, 3, 0.5, 2, 2),           # 3228 and 1615
    (40, 128, 5, 24, 25, 77, 0.34, 2, 3),        # 3077 and 1020
    (48, 6144, 5, 21, 40, 3, 0.75, 2, 2),        # 4203 and 3200
    (40, 1088, 6, 18, 34, 3, 0.75, 2, 3),        # 3675 and 3078
    (64, 2048, 7, 34, 19, 3, 1.0, 2, 3),         # 4525 and 4522: out-projection and FFN2 cut along k
]


def block_config(heads, ffn, frames, height, width, n_text, ratio, patch_h, patch_w, flags=0, fp32=True):
    return get_config("tiny", n_layers=1, n_shallow=1, hidden=64 * heads, n_heads=heads, head_dim=64, ffn_dim=ffn, frames=frames,
                      height=height, width=width, n_text=n_text, ratio=ratio, patch_h=patch_h, patch_w=patch_w,
                      block_flags=flags, resid_fp32=fp32)


def weights(cfg, gen, most=1088, qkv_std=0.04):
    """Drawn with standard deviations that keep what a projection of up to `most` channels (FFN2: 4 x as many) gives
    at the size it has there, so that the absolute tolerance means the same at every width."""
    d, f = cfg.hidden, cfg.ffn_dim
    s, s2 = min(1.0, math.sqrt(most / d)), min(1.0, math.sqrt(4 * most / f))

    def normal(*shape, std=0.02, mean=0.0):
        return (torch.randn(*shape, generator=gen, device="cuda") * std + mean).to(torch.bfloat16)

    w = {"w_qkv": normal(3 * d, d, std=qkv_std * s), "b_qkv": normal(3 * d), "w_o": normal(d, d, std=0.02 * s), "b_o": normal(d),
         "w_ff1": normal(f, d, std=0.02 * s), "b_ff1": normal(f), "w_ff2": normal(d, f, std=0.02 * s2), "b_ff2": normal(d),
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


def run_block(cfg, qkv_std=0.04):
    """One layer of `cfg` in full, then refreshed on the rows the selection picks, against float64 torch: K, V^T, S and x."""
    d, fp32 = cfg.hidden, cfg.resid_fp32
    print(f"[case] {cfg.n_tokens} rows, hidden {d}, ffn {cfg.ffn_dim}, flags {cfg.block_flags}, fp32 {fp32}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    cache = B.HeroCache(B.make_config(cfg))
    w = weights(cfg, gen, qkv_std=qkv_std)
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
