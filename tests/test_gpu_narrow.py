"""Models of at most 256 channels, whose QKV and FFN1 kernels normalise their rows themselves, and the first
width past that: one block in full and refreshed, against the same block in float64 torch."""
import pytest
import torch

from paper_2508_17588_amd import binding as B
from torch_block import run_block, weights
from workloads import BLOCK_ADALN, get_config

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags,fp32", [(0, True), (BLOCK_ADALN, False)])
@pytest.mark.parametrize("heads,frames,height,width,n_text", [
    (1, 1, 4, 5, 1),          # 64 channels, 21 rows: half the lanes of a row idle, most of a tile's rows missing
    (2, 2, 7, 9, 3),          # 128 channels, 129 rows: one row in the last tile
    (3, 2, 10, 15, 26),       # 192 channels: a quarter of a row's lanes idle, Q / K / V boundaries on tile edges
    (4, 2, 10, 15, 26),       # 256 channels, 16 waves
    (4, 5, 16, 19, 77),       # 256 channels, more than 256 tiles: eight waves
    (5, 2, 10, 15, 26),       # 320 channels: LayerNorm by itself
])
def test_block_of_a_narrow_model(heads, frames, height, width, n_text, flags, fp32):
    d = heads * 64
    run_block(get_config("tiny", n_layers=1, n_shallow=1, hidden=d, n_heads=heads, head_dim=64, ffn_dim=4 * d, frames=frames,
                         height=height, width=width, n_text=n_text, block_flags=flags, resid_fp32=fp32))


@pytest.mark.parametrize("flags,fp32", [(0, True), (BLOCK_ADALN, False)])
@pytest.mark.parametrize("heads,frames,height,width,n_text", [
    (1, 1, 3, 5, 0),          # 15 rows: less than one workgroup's
    (2, 1, 3, 5, 1),          # 16, and some listed ones
    (3, 1, 3, 5, 2),          # 17
    (1, 3, 11, 31, 1),        # 1024 rows: FFN channels shared by four workgroups
    (4, 3, 11, 31, 2),        # 1025: by two
    (2, 1, 23, 89, 1),        # 2048
    (4, 1, 23, 89, 2),        # 2049: not shared
    (4, 1, 63, 65, 1),        # 4096: one round
    (3, 1, 63, 65, 2),        # 4097: the three separate kernels
    (3, 1, 64, 97, 1),        # 6209: two rounds
    (2, 1, 64, 97, 3),        # at 128 channels: any number
    (4, 1, 64, 128, 1),       # 8193: separate kernels again (listed rows: one)
])
def test_rows_from_attention_to_residual_in_one_kernel(heads, frames, height, width, n_text, flags, fp32):
    d = heads * 64
    run_block(get_config("tiny", n_layers=1, n_shallow=1, hidden=d, n_heads=heads, head_dim=64, ffn_dim=4 * d, frames=frames,
                         height=height, width=width, n_text=n_text, block_flags=flags, resid_fp32=fp32))


def test_shared_ffn_channels_add_up_the_same_whoever_arrives_last():
    cfg = get_config("tiny", n_layers=1, n_shallow=1, hidden=256, n_heads=4, head_dim=64, ffn_dim=1024, frames=1, height=31,
                     width=33, n_text=1)                                  # 1024 rows: 256 workgroups
    gen = torch.Generator(device="cuda")
    gen.manual_seed(11)
    cache = B.HeroCache(B.make_config(cfg))
    cache.hero_set_layer_weights(0, weights(cfg, gen))
    x0 = torch.randn(cfg.n_tokens, 256, generator=gen, device="cuda")
    first = None
    for _ in range(20):
        x = x0.clone()
        cache.hero_full_layer(0, x)
        got = torch.cat([x, cache.hero_cache_view(0, B.VIEW_S_CUR).float()])
        first = got if first is None else first
        assert torch.equal(got, first)
    cache.close()
