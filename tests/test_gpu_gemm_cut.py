"""Layers whose GEMMs are cut along k between workgroups that add their parts up themselves: every kind of tile, whole
rounds before the cut one or none, remainders of rows and columns, all rows and listed ones, against float64 torch; and
the same bits on every call, whichever workgroup arrives last."""
import pytest
import torch

from paper_2508_17588_amd import binding as B
from torch_block import run_block, weights
from workloads import BLOCK_ADALN, get_config

pytestmark = pytest.mark.gpu

OUT, FFN1, FFN2 = B.ROUTE_OUT, B.ROUTE_FFN1, B.ROUTE_FFN2


def every(*tile):
    return {OUT: tile, FFN1: tile, FFN2: tile}


# Heads of 64 channels, FFN width, height, width, text rows; the tiles of those GEMMs that are cut, and into how many chunks, on
# all rows and on all but the text rows.  Between them every kind of tile that a layer cuts (tests/test_routes.py).
SHAPES = [
    (12, 3072, 30, 50, 1, {FFN2: (128, 128, 3)}, {FFN2: (128, 128, 3)}),                  # 1501 rows
    (33, 8448, 7, 8, 4, {FFN2: (64, 64, 4)}, {FFN2: (64, 64, 4)}),                        # 60: one row tile
    (48, 12288, 8, 41, 2, {OUT: (128, 128, 3), FFN2: (128, 128, 3)}, {OUT: (128, 128, 3), FFN2: (128, 128, 3)}),     # 330
    (33, 8448, 25, 40, 1, {FFN2: (128, 192, 2)}, {FFN2: (128, 192, 2)}),                  # 1001
    (31, 7936, 32, 64, 1, {FFN2: (192, 192, 2)}, {}),                                     # 2049: columns end inside a tile
    (45, 11520, 20, 35, 1, {FFN2: (192, 192, 4)}, {FFN2: (192, 192, 4)}),                 # 701
    (49, 12544, 20, 35, 1, {FFN2: (256, 128, 3)}, {FFN2: (256, 128, 3)}),                 # 701
    (47, 12032, 48, 64, 5, {FFN1: (256, 256, 2), FFN2: (192, 192, 7)}, {}),               # 3077: a round of whole tiles, then 16 in 7
    (24, 6144, 6, 7, 3, {FFN2: (64, 64, 4)}, {FFN2: (64, 64, 4)}),                        # 45
    (31, 7936, 8, 10, 4, {FFN2: (64, 64, 4)}, {FFN2: (64, 64, 4)}),                       # 84: columns end inside the last group of eight tiles
    (17, 4352, 12, 12, 6, {FFN2: (64, 64, 3)}, {FFN2: (64, 64, 3)}),                      # 150
    (48, 3072, 7, 7, 1, every(64, 64, 3), every(64, 64, 3)),                              # 50
    (48, 9216, 9, 10, 3, {FFN1: (128, 128, 3), FFN2: (64, 64, 2)}, {FFN1: (128, 128, 3), FFN2: (64, 64, 2)}),        # 93: one row tile of 128
    (52, 3328, 18, 18, 9, every(128, 128, 2), every(128, 128, 2)),                        # 333
    (42, 2688, 77, 92, 6, every(192, 192, 3), every(192, 192, 3)),                        # 7090: two rounds of whole tiles first
    (128, 9216, 14, 15, 3, {OUT: (128, 128, 2), FFN1: (128, 192, 2), FFN2: (128, 128, 2)},
     {OUT: (128, 128, 2), FFN1: (128, 192, 2), FFN2: (128, 128, 2)}),                     # 213
    (128, 16384, 33, 38, 2, {FFN1: (256, 128, 2)}, {FFN1: (256, 128, 2)}),                # 1256
]


def config(heads, ffn, height, width, n_text, cuts, listed_cuts, flags=0, fp32=True):
    """The shape's configuration, of which the library cuts what the shape says."""
    d = heads * 64
    cfg = get_config("tiny", n_layers=1, n_shallow=1, hidden=d, n_heads=heads, head_dim=64, ffn_dim=ffn, frames=1,
                     height=height, width=width, n_text=n_text, ratio=1.0, block_flags=flags, resid_fp32=fp32)
    for want, rows, listed in ((cuts, cfg.n_tokens, False), (listed_cuts, height * width, True)):
        routes = {what: B.hero_layer_route(B.make_config(cfg), rows, what, listed) for what in (OUT, FFN1, FFN2)}
        assert {what: r[1:] for what, r in routes.items() if r[3] > 1} == want, (cfg.n_tokens, listed, routes)
    return cfg


@pytest.mark.parametrize("shape", SHAPES)
def test_cut_layers(shape):
    run_block(config(*shape))


@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[3], SHAPES[9], SHAPES[11], SHAPES[13]])
def test_cut_layers_modulated_bf16_stream(shape):
    run_block(config(*shape, flags=BLOCK_ADALN, fp32=False))


@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[2], SHAPES[5], SHAPES[7], SHAPES[8], SHAPES[11], SHAPES[12]])
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
