"""Per-layer extrapolation, whose even layers walk the arrays from the end: the same bits as hero_axpy_features, which walks them
from the start, with whole groups of eight blocks and with a ragged last block."""
import pytest
import torch

from paper_2508_17588_amd import binding as B
from torch_block import weights
from workloads import get_config

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tokens,hidden,fp32,generations", [
    (45, 64, True, 2),            # 360 chunks of 8 elements: two blocks of a group of eight
    (512, 1024, True, 2),         # 256 whole blocks
    (1031, 192, True, 1),         # 97 blocks, the last one ragged; one generation: no previous features to read
    (1031, 192, False, 2),
])
def test_either_direction_gives_the_same_bits(tokens, hidden, fp32, generations):
    print(f"[case] {tokens} x {hidden}, fp32 {fp32}, {generations} generations", flush=True)
    cfg = get_config("tiny", n_layers=2, n_shallow=0, interval=3, hidden=hidden, n_heads=hidden // 64, head_dim=64, ffn_dim=64,
                     frames=1, height=1, width=tokens, n_text=0, resid_fp32=fp32)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(2)
    cache = B.HeroCache(B.make_config(cfg))
    x0 = torch.randn(tokens, hidden, generator=gen, device="cuda").to(torch.float32 if fp32 else torch.bfloat16)
    for l in range(2):
        cache.hero_set_layer_weights(l, weights(cfg, gen))
        for g in range(generations):
            cache.hero_full_layer(l, x0.flip(0).contiguous() if g else x0.clone())
    for l in range(2):
        got, want = x0.clone(), x0.clone()
        cache.hero_extrapolate_layer(l, got, 1)
        prev = cache.hero_cache_view(l, B.VIEW_S_PREV) if generations > 1 else None
        B.hero_axpy_features(want, cache.hero_cache_view(l, B.VIEW_S_CUR), prev, 1 / 3)
        assert torch.equal(got, want) and not torch.equal(got, x0)
    cache.close()
