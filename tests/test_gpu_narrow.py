"""Models of at most 256 channels, whose QKV and FFN1 kernels normalise their rows themselves, or whose rows one kernel takes
from the attention output to the residual add where the FFN is four times as wide, and the first width past that: one
block in full and refreshed, against the same block in float64 torch."""
import pytest
import torch

from paper_2508_17588_amd import binding as B
from torch_block import run_block, weights
from workloads import BLOCK_ADALN, get_config

pytestmark = pytest.mark.gpu


def config(heads, ffn, frames, height, width, n_text, flags=0, fp32=True):
    d = heads * 64
    return get_config("tiny", n_layers=1, n_shallow=1, hidden=d, n_heads=heads, head_dim=64, ffn_dim=ffn, frames=frames,
                      height=height, width=width, n_text=n_text, block_flags=flags, resid_fp32=fp32)


def forms(cfg, listed=False):
    """The forms of the four GEMMs of a layer, on all rows or on the selected ones."""
    c = B.make_config(cfg)
    rows = B.hero_num_selected(c) if listed else cfg.n_tokens
    return [B.hero_layer_route(c, rows, what, listed)[0] for what in (B.ROUTE_QKV, B.ROUTE_OUT, B.ROUTE_FFN1, B.ROUTE_FFN2)]


NORMALISING = [               # heads, frames, height, width, text rows
    (1, 1, 4, 5, 1),          # 64 channels, 21 rows: half the lanes of a row idle, most of a tile's rows missing
    (2, 2, 7, 9, 3),          # 128 channels, 129 rows: one row in the last tile
    (3, 2, 10, 15, 26),       # 192 channels: a quarter of a row's lanes idle, Q / K / V boundaries on tile edges
    (4, 2, 10, 15, 26),       # 256 channels, 16 waves
    (4, 5, 16, 19, 77),       # 256 channels, more than 256 tiles: eight waves
    (5, 2, 10, 15, 26),       # 320 channels: LayerNorm by itself
]


@pytest.mark.parametrize("flags,fp32", [(0, True), (BLOCK_ADALN, False)])
@pytest.mark.parametrize("widths", [3, 4])          # FFN channels for each of the stream: three kernels, or one
@pytest.mark.parametrize("heads,frames,height,width,n_text", NORMALISING)
def test_block_of_a_narrow_model(heads, frames, height, width, n_text, widths, flags, fp32):
    cfg = config(heads, widths * heads * 64, frames, height, width, n_text, flags, fp32)
    for listed in (False, True):
        if heads > 4:
            want = [B.FORM_GEMM] * 4
        elif widths == 4:
            want = [B.FORM_LN_GEMM, B.FORM_TAIL, B.FORM_TAIL, B.FORM_TAIL]
        else:
            want = [B.FORM_LN_GEMM, B.FORM_GEMM, B.FORM_LN_GEMM, B.FORM_GEMM]
        assert forms(cfg, listed) == want
    run_block(cfg)


ONE_KERNEL = [                # heads, frames, height, width, text rows; workgroups that share a block's FFN channels (0: another kernel), the same on listed rows
    (1, 1, 3, 5, 0, 4, 4),          # 15 rows: less than one workgroup's
    (2, 1, 3, 5, 1, 4, 4),          # 16, and some listed ones
    (3, 1, 3, 5, 2, 4, 4),          # 17
    (1, 3, 11, 31, 1, 4, 4),        # 1024 rows: FFN channels shared by four workgroups
    (4, 3, 11, 31, 2, 2, 4),        # 1025: by two
    (2, 1, 23, 89, 1, 2, 4),        # 2048
    (4, 1, 23, 89, 2, 1, 4),        # 2049: not shared
    (4, 1, 63, 65, 1, 1, 2),        # 4096: one round
    (3, 1, 63, 65, 2, 0, 2),        # 4097: the three separate kernels
    (3, 1, 64, 97, 1, 1, 2),        # 6209: two rounds
    (2, 1, 64, 97, 3, 1, 2),        # at 128 channels: any number
    (4, 1, 64, 128, 1, 0, 2),       # 8193: separate kernels again (listed rows: one)
    (1, 1, 63, 65, 1, 1, 2),        # 4096 rows of 64 channels
    (1, 1, 23, 89, 1, 2, 4),        # 2048
    (3, 1, 23, 89, 1, 2, 4),        # 2048 rows of 192 channels
    (1, 2, 64, 80, 3, 1, 1),        # listed rows not shared either: more than 2048 of them
    (2, 2, 64, 80, 3, 1, 1),
    (3, 2, 64, 80, 3, 0, 1),
    (4, 2, 64, 80, 3, 0, 1),
]


@pytest.mark.parametrize("flags,fp32", [(0, True), (BLOCK_ADALN, False)])
@pytest.mark.parametrize("heads,frames,height,width,n_text,shared,listed_shared", ONE_KERNEL)
def test_rows_from_attention_to_residual_in_one_kernel(heads, frames, height, width, n_text, shared, listed_shared, flags, fp32):
    cfg = config(heads, 4 * heads * 64, frames, height, width, n_text, flags, fp32)
    c = B.make_config(cfg)
    for rows, listed, want in ((cfg.n_tokens, False, shared), (B.hero_num_selected(c), True, listed_shared)):
        for what in (B.ROUTE_OUT, B.ROUTE_FFN1, B.ROUTE_FFN2):
            form, *route = B.hero_layer_route(c, rows, what, listed)
            assert (form == B.FORM_TAIL) == (want > 0)
            assert want == 0 or route == [16, heads * 64, want]
    run_block(cfg)


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
