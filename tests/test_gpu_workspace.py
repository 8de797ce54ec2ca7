"""A workspace that other work has written to between the calls: what a layer counts on from one call to the next lies in
the cache buffer."""
import pytest
import torch

from paper_2508_17588_amd import binding as B
from torch_block import weights
from workloads import get_config

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,height,width", [
    (4, 18, 18),          # FFN channels shared by workgroups that count their arrivals
    (24, 6, 7),           # tiles cut along k, likewise
    (47, 48, 64),         # the same after a round of whole tiles
])
def test_layers_do_not_depend_on_what_the_workspace_holds(heads, height, width):
    d = heads * 64
    print(f"[case] hidden {d}, {height * width + 3} rows", flush=True)
    cfg = get_config("tiny", n_layers=1, n_shallow=1, hidden=d, n_heads=heads, head_dim=64, ffn_dim=4 * d, frames=1,
                     height=height, width=width, n_text=3, ratio=0.34)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    cache = B.HeroCache(B.make_config(cfg))
    cache.hero_set_layer_weights(0, weights(cfg, gen))
    x0 = torch.randn(cfg.n_tokens, d, generator=gen, device="cuda")
    idx = torch.zeros(cfg.n_tokens, dtype=torch.int32, device="cuda")

    def layers(fill):
        out = []
        cache.hero_cache_reset()
        for call in ("full", "refresh"):
            x = x0.clone()
            if fill is not None:
                cache.ws_buf.fill_(fill)          # (0x7f7f is a large finite bf16, 0x7f7f7f7f a large finite fp32)
            if call == "full":
                cache.hero_full_layer(0, x)
            else:
                n = cache.hero_select(1, idx)
                if fill is not None:
                    cache.ws_buf.fill_(fill)
                cache.hero_refresh_layer(0, x, idx, n)
            out += [x, cache.hero_cache_view(0, B.VIEW_S_CUR).clone()]
        return out

    want = layers(None)
    for fill in (0x7f, 0x01, 0x00):
        for got, w in zip(layers(fill), want):
            assert torch.equal(got, w), f"workspace of {fill:#x}"
    cache.close()
