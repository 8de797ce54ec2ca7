"""Layers whose GEMMs are cut along k between workgroups that add their parts up themselves: every kind of tile, whole
rounds before the cut one or none, remainders of rows and columns, all rows and listed ones, against float64 torch; and
the same bits on every call, whichever workgroup arrives last."""
import pytest
import torch

from paper_2508_17588_amd import binding as B
from torch_block import run_block, weights
from workloads import BLOCK_ADALN, get_config

pytestmark = pytest.mark.gpu

SHAPES = [                     # heads of 64 channels, height, width, text rows
    (12, 30, 50, 1),           # 1501 rows: FFN2 128 x 128 in 3
    (33, 7, 8, 4),             # 60: 128 x 128 in 6, one row tile
    (48, 8, 41, 2),            # 330: out-projection and FFN2 128 x 128 in 3
    (33, 25, 40, 1),           # 1001: 128 x 192 in 2
    (31, 32, 64, 1),           # 2049: 192 x 192 in 2, columns end inside a tile
    (45, 20, 35, 1),           # 701: 192 x 192 in 4
    (49, 20, 35, 1),           # 701: 256 x 128 in 3
    (47, 48, 64, 5),           # 3077: 192 x 192, a round of whole tiles, then 16 tiles in 7
    (24, 6, 7, 3),             # 45: 64 x 64 in 6
    (31, 8, 10, 4),            # 84: 64 x 64 in 4, columns end inside the last group of eight tiles
    (17, 12, 12, 6),           # 150: 64 x 64
]


def config(heads, height, width, n_text, flags=0, fp32=True):
    d = heads * 64
    return get_config("tiny", n_layers=1, n_shallow=1, hidden=d, n_heads=heads, head_dim=64, ffn_dim=4 * d, frames=1,
                      height=height, width=width, n_text=n_text, ratio=1.0, block_flags=flags, resid_fp32=fp32)


@pytest.mark.parametrize("shape", SHAPES)
def test_cut_layers(shape):
    run_block(config(*shape))


@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[3], SHAPES[9]])
def test_cut_layers_modulated_bf16_stream(shape):
    run_block(config(*shape, flags=BLOCK_ADALN, fp32=False))


@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[2], SHAPES[5], SHAPES[7], SHAPES[8]])
def test_every_call_gives_the_same_bits(shape):
    cfg = config(*shape)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    cache = B.HeroCache(B.make_config(cfg))
    cache.hero_set_layer_weights(0, weights(cfg, gen))
    x0 = torch.randn(cfg.n_tokens, cfg.hidden, generator=gen, device="cuda")
    first = None
    for _ in range(10):
        x = x0.clone()
        cache.hero_full_layer(0, x)
        got = torch.cat([x, cache.hero_cache_view(0, B.VIEW_S_CUR).float()])
        first = got if first is None else first
        assert torch.equal(got, first)
    cache.close()
