"""Models of at most 256 channels, whose QKV and FFN1 kernels normalise their rows themselves, and the first
width past that: one block in full and refreshed, against the same block in float64 torch."""
import pytest

from torch_block import run_block
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
