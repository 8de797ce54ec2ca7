"""A cached step of a model with one deep layer, whose extrapolation rides in the pass that ends the step: with one
generation (no difference to extrapolate) and two, odd row counts, both residual streams, against float64."""
import pytest
import torch

from paper_2508_17588_amd import binding as B
from workloads import get_config
from torch_block import weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp32", [True, False])
@pytest.mark.parametrize("n_shallow", [1, 2])
@pytest.mark.parametrize("heads,height,width", [(1, 3, 5), (9, 7, 11)])
def test_cached_step_adds_the_deep_layer(heads, height, width, n_shallow, fp32):
    d = heads * 64
    cfg = get_config("tiny", n_layers=n_shallow + 1, n_shallow=n_shallow, interval=3, hidden=d, n_heads=heads,
                     head_dim=64, ffn_dim=4 * d, frames=2, height=height, width=width, n_text=5, resid_fp32=fp32)
    print(f"[case] {cfg.n_tokens} rows, hidden {d}, {n_shallow} shallow, fp32 {fp32}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    cache = B.HeroCache(B.make_config(cfg))
    for l in range(cfg.n_layers):
        cache.hero_set_layer_weights(l, weights(cfg, gen))
    for step in range(6):
        x = torch.randn(cfg.n_tokens, d, generator=gen, device="cuda").to(torch.float32 if fp32 else torch.bfloat16)
        x0 = x.double()
        cache.hero_step(x, step)
        if step % 3 == 0:
            continue
        torch.cuda.synchronize()
        parts = [cache.hero_cache_view(l, B.VIEW_S_CUR).double() for l in range(cfg.n_layers)]
        prev = cache.hero_cache_view(n_shallow, B.VIEW_S_PREV).double() if step > 3 else parts[-1]
        want = x0 + sum(parts) + (parts[-1] - prev) * (step % 3 / 3)
        size = x0.abs() + sum(p.abs() for p in parts) + parts[-1].abs() + prev.abs()
        # refreshed rows are rounded once a shallow layer and once at the end, each to the stream's type
        bound = (n_shallow + 5) * (2.0 ** -24 if fp32 else 2.0 ** -9) * size
        err = (x.double() - want).abs()
        assert bool((err <= bound).all()), f"step {step}: off by {float((err - bound).max())}"
    cache.close()
