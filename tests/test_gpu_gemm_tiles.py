"""The GEMMs at ragged sizes.  One block run in full and then refreshed on listed rows, against the same block in
float64 torch: first at the shapes between which every epilogue takes every kind of tile (64 x 64, 128 x 128,
128 x 192, 192 x 192, 256 x 128, 256 x 256), on all rows and on listed ones, gated with a bf16 residual stream and
plain with an fp32 one; then at a few more.  And hero_linear: the kinds, few stages of the largest tiles, tiles cut
along k.  Which kernel runs is asserted, not assumed.
"""
import pytest
import torch

from paper_2508_17588_amd import binding as B
from workloads import BLOCK_ADALN, get_config
from hero_testlib import assert_close, to_host_f64
from torch_block import BLOCKS, block_config, run_block

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags,fp32", [(0, True), (BLOCK_ADALN, False)])
@pytest.mark.parametrize("shape", BLOCKS, ids=lambda s: "-".join(map(str, s)))
def test_block_with_every_tile_kind(shape, flags, fp32):
    # Scores of standard deviation 1.  An attention output over thousands of keys is as small as the sum of its rounding
    # errors is: with u = 1.1e-3 for one bf16 rounding, about u sqrt(5 + 2 sigma^2) of itself (v, the probabilities, the
    # output, its projection and S are rounded; q and k move each score by sigma u sqrt(2)), 2.9e-3 at sigma = 1 and more
    # than 3.7e-3 at 1.7 (the standard deviation in the other tests), where a narrow FFN adds little to hide it.
    run_block(block_config(*shape, flags=flags, fp32=fp32), qkv_std=0.03)


@pytest.mark.parametrize("heads,frames,height,width,n_text,flags,fp32", [
    (1, 1, 7, 7, 16, 0, True),               # hidden 64: one stage along k, Q, K and V inside one tile
    (7, 3, 9, 11, 3, BLOCK_ADALN, False),    # 300 rows
    (17, 3, 12, 19, 17, BLOCK_ADALN, True),  # 701 rows
    (16, 4, 17, 19, 8, 0, False),            # 1300 rows
    (17, 5, 17, 23, 77, BLOCK_ADALN, True),  # 2032 rows
    (17, 4, 23, 27, 16, 0, False),           # 2500 rows
])
def test_block_at_ragged_sizes(heads, frames, height, width, n_text, flags, fp32):
    d = heads * 64
    run_block(get_config("tiny", n_layers=1, n_shallow=1, hidden=d, n_heads=heads, head_dim=64, ffn_dim=4 * d, frames=frames,
                         height=height, width=width, n_text=n_text, block_flags=flags, resid_fp32=fp32))


def linear(m, n, k, act, scratch_mib=0):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m)
    a = torch.randn(m, k, generator=gen, device="cuda").to(torch.bfloat16)
    w = (torch.randn(n, k, generator=gen, device="cuda") * min(0.02, 1 / k ** 0.5)).to(torch.bfloat16)
    bias = torch.randn(n, generator=gen, device="cuda").to(torch.bfloat16)
    guard = torch.full((m + 1, n), 7.0, dtype=torch.bfloat16, device="cuda")     # the row past the end stays as it is
    want = a.double() @ w.double().T + bias.double()
    if act:
        want = torch.nn.functional.gelu(want, approximate="tanh")
    if scratch_mib:
        scratch = torch.full((scratch_mib << 18,), float("nan"), dtype=torch.float32, device="cuda")
        B.hero_linear_scratch(a, w, bias, guard, scratch, act)
    else:
        B.hero_linear(a, w, bias, guard, act)
    torch.cuda.synchronize()
    assert bool((guard[m] == 7.0).all())
    assert_close(to_host_f64(guard[:m]), want.cpu().numpy(), f"linear {m}x{n}x{k} act {act}")


@pytest.mark.parametrize("m,n,k,tile", [
    (1, 64, 64, (64, 64)), (65, 192, 320, (64, 64)), (326, 256, 1024, (64, 64)), (691, 3072, 1024, (128, 128)),
    (1755, 3072, 3072, (128, 192)), (2925, 3072, 1024, (192, 192)), (2032, 4160, 1024, (192, 192)),
    (1987, 1984, 1088, (128, 128)), (4001, 2048, 64, (256, 128)),
    # the largest tiles with 1, 5 and 7 stages of 64 (the loop over stages is unrolled six times, the activation ring is
    # three slots deep)
    (7131, 1216, 64, (256, 256)), (7131, 1216, 320, (256, 256)), (7131, 1216, 448, (256, 256)),
])
def test_linear_tile_edges(m, n, k, tile):
    print(f"[case] linear {m} x {n} x {k}", flush=True)
    for act, what in ((0, B.ROUTE_PLAIN), (1, B.ROUTE_GELU)):
        assert B.hero_linear_route(m, n, k, what)[:2] == tile
        linear(m, n, k, act)


@pytest.mark.parametrize("m,n,k,act,scratch_mib,chunks", [
    (2470, 6592, 6144, 1, 64, 6),        # 260 tiles: 256 whole, 4 (of 8 slots) cut in six
    (2726, 6592, 2048, 0, 64, 2),        # 286 tiles
    (4774, 6848, 6144, 0, 64, 6),        # 513 tiles: two rounds and a tile
    (4774, 6848, 6144, 0, 8, 4),         # scratch for four chunks of a slot only
    (4774, 6848, 2048, 1, 1, 1),         # for none
])
def test_linear_cut_along_k(m, n, k, act, scratch_mib, chunks):
    print(f"[case] linear {m} x {n} x {k} with {scratch_mib} MiB", flush=True)
    route = B.hero_linear_route(m, n, k, B.ROUTE_GELU if act else B.ROUTE_PLAIN, False, scratch_mib << 20)
    assert route[:3] == (256, 256, chunks)
    linear(m, n, k, act, scratch_mib)
