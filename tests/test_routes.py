"""Which kernel a problem goes to (host only)."""
import random

import pytest

import test_gpu_gemm_cut
import test_gpu_narrow
from paper_2508_17588_amd import binding as B
from torch_block import BLOCKS, block_config
from workloads import get_config

MIB = 1 << 20
TILES = {(64, 64), (128, 128), (128, 192), (192, 192), (256, 128), (256, 256)}


@pytest.mark.parametrize("what", [B.ROUTE_PLAIN, B.ROUTE_GELU, B.ROUTE_QKV, B.ROUTE_OUT, B.ROUTE_FFN1, B.ROUTE_FFN2])
@pytest.mark.parametrize("listed", [False, True])
def test_linear_routes_over_the_range(what, listed):
    seen = set()
    for hidden in (64, 192, 448, 1024, 1920, 3072, 8192):
        for m in (1, 63, 65, 300, 691, 1755, 2925, 4485, 17776):
            n = 3 * hidden if what == B.ROUTE_QKV else hidden
            for scratch in (0, MIB, 128 * MIB):
                tm, tn, chunks, normalises = B.hero_linear_route(m, n, hidden, what, listed, scratch)
                assert (tm, tn) in TILES and 1 <= chunks <= 8
                # only 256 x 256 tiles are cut, only with scratch that holds a block of every chunk, never a QKV projection
                assert chunks == 1 or ((tm, tn) == (256, 256) and scratch >= chunks * 256 * 256 * 4 and what != B.ROUTE_QKV)
                # a wave's columns of a 256 x 256 tile lie inside one of Q, K and V
                assert what != B.ROUTE_QKV or hidden % 128 == 0 or (tm, tn) != (256, 256)
                assert not normalises or (hidden <= 256 and what in (B.ROUTE_QKV, B.ROUTE_FFN1) and (tm, tn) == (64, 64))
                seen.add((tm, tn))
    assert len(seen) >= 4


def test_attention_routes_over_the_range():
    for r in (1, 65, 300, 1755, 4485, 17776):
        for n_keys in (1, 90, 2032, 17776):
            for heads in (1, 4, 16, 48):
                few = 32 if (r + 31) // 32 * heads <= 256 else 64          # one workgroup of 32 queries a CU
                assert B.hero_attention_route(r, n_keys, heads, 32, 128 * MIB) == (few, 1)
                queries, ranges = B.hero_attention_route(r, n_keys, heads, 64, 128 * MIB)
                assert queries in (few, 256) and 1 <= ranges <= 16 and (queries == 256 or ranges == 1)
                assert B.hero_attention_route(r, n_keys, heads, 64, 0)[1] == 1
    assert B.hero_attention_route(4485, 17776, 48, 64, 128 * MIB) == (256, 4)


def test_routes_refuse_what_the_calls_refuse():
    for args in ((0, 64, 64), (1, 64, 65), (1, 65, 64), (1, 64, 64, 6), (1, 128, 64, B.ROUTE_QKV), (699_051, 256, 3072)):
        with pytest.raises(B.HeroError):
            B.hero_linear_route(*args)
    for args in ((1, 1, 1, 48), (1, 0, 1, 64), (1, 699_100, 48, 64)):
        with pytest.raises(B.HeroError):
            B.hero_attention_route(*args)


@pytest.mark.parametrize("m,n,k,what,listed,tile", [
    # as measured (kernel times of every kind): what had gone to another kind for less than the expected times are good for
    (4485, 12288, 3072, B.ROUTE_FFN1, True, (256, 256)),      # 296 us; 192 x 192 303
    (17776, 1920, 7680, B.ROUTE_FFN2, False, (256, 256)),     # 530 us; 192 x 192 549
    # listed rows whose V^T columns were not part of the expected time
    (4485, 1536, 512, B.ROUTE_QKV, True, (128, 128)),         # 22.7 us; 256 x 128 25.9
    (691, 1536, 512, B.ROUTE_QKV, True, (64, 64)),            # 12.1 us; 128 x 128 15.3
    (2925, 2304, 768, B.ROUTE_QKV, True, (128, 128)),         # 26.4 us; 256 x 128 29.3
    # and what the smaller tiles are there for
    (2925, 3072, 12288, B.ROUTE_FFN2, True, (192, 192)),      # 194 us; 256 x 256 241
    (691, 1024, 4096, B.ROUTE_FFN2, True, (64, 64)),          # 16.2 us; 128 x 128 28.3
    (17776, 1920, 1920, B.ROUTE_OUT, False, (192, 192)),      # 132 us; 256 x 256 140
])
def test_measured_choices(m, n, k, what, listed, tile):
    assert B.hero_linear_route(m, n, k, what, listed, 128 * MIB)[:2] == tile


@pytest.mark.parametrize("m,hidden,ffn,qkv,ffn1", [
    # kernels by themselves: four layers, us, with FFN1 normalising or not as noted
    (326, 128, 512, True, True),
    (17576, 64, 4096, True, False),          # 769; normalising 927
    (17576, 128, 512, True, True),           # 771; apart 807
    (17576, 128, 8192, True, False),         # 1546; normalising 1889
    (8126, 256, 1024, False, False),         # 510; both normalising 549
    (1306, 256, 4096, True, False),          # 214; normalising 244
    (1306, 256, 1024, True, True),           # 165; apart 182
    (90, 320, 1280, False, False),
])
def test_measured_choices_of_narrow_models(m, hidden, ffn, qkv, ffn1):
    assert bool(B.hero_linear_route(m, 3 * hidden, hidden, B.ROUTE_QKV)[3]) == qkv
    assert bool(B.hero_linear_route(m, ffn, hidden, B.ROUTE_FFN1)[3]) == ffn1


def layer_config(tokens, hidden, ffn):
    return B.make_config(get_config("tiny", n_layers=1, n_shallow=1, hidden=hidden, n_heads=hidden // 64, head_dim=64, ffn_dim=ffn,
                                    frames=1, height=1, width=tokens, n_text=0))


@pytest.mark.parametrize("m,hidden,ffn,qkv,ffn1", [
    # what a layer launches: with an FFN four times as wide one kernel takes the rows to the residual add where that is faster
    (326, 128, 512, B.FORM_LN_GEMM, B.FORM_TAIL),
    (33000, 64, 256, B.FORM_LN_GEMM, B.FORM_TAIL),           # four layers, us: 1195; three kernels 1287
    (33000, 128, 512, B.FORM_LN_GEMM, B.FORM_TAIL),          # 2300; 2396
    (8000, 256, 1024, B.FORM_GEMM, B.FORM_TAIL),          # 507; 522
    (10000, 256, 1024, B.FORM_GEMM, B.FORM_GEMM),         # 683; one kernel 712
    (5000, 192, 768, B.FORM_LN_GEMM, B.FORM_GEMM),           # 269; 275
    (6500, 192, 768, B.FORM_GEMM, B.FORM_TAIL),           # 348; three kernels 384
    (33000, 192, 768, B.FORM_GEMM, B.FORM_GEMM),          # 3428; one kernel 3531
    (1306, 256, 1024, B.FORM_LN_GEMM, B.FORM_TAIL),
    # other widths: as the kernels by themselves
    (17576, 64, 4096, B.FORM_LN_GEMM, B.FORM_GEMM),
    (326, 128, 256, B.FORM_LN_GEMM, B.FORM_LN_GEMM),
    (1306, 256, 4096, B.FORM_LN_GEMM, B.FORM_GEMM),
    (90, 320, 1280, B.FORM_GEMM, B.FORM_GEMM),
])
def test_forms_of_the_layers_of_narrow_models(m, hidden, ffn, qkv, ffn1):
    c = layer_config(m, hidden, ffn)
    assert [B.hero_layer_route(c, m, what)[0] for what in (B.ROUTE_QKV, B.ROUTE_FFN1)] == [qkv, ffn1]
    for what in (B.ROUTE_OUT, B.ROUTE_FFN2):
        assert B.hero_layer_route(c, m, what)[0] == (B.FORM_TAIL if ffn1 == B.FORM_TAIL else B.FORM_GEMM)


@pytest.mark.parametrize("m,hidden,ffn,what,route", [
    # kernel times in a layer, us, and without the cut
    (45, 1536, 6144, B.ROUTE_FFN2, (64, 64, 4)),          # 12.7; 19.8
    (84, 1920, 7680, B.ROUTE_FFN2, (64, 64, 4)),          # 14.4; 24.4
    (700, 1536, 6144, B.ROUTE_FFN2, (128, 128, 3)),       # 26.7; 41.0
    (1500, 3072, 12288, B.ROUTE_FFN2, (192, 192, 2)),     # 117; 148 (128 x 192)
])
def test_measured_cuts_of_a_layer(m, hidden, ffn, what, route):
    assert B.hero_layer_route(layer_config(m, hidden, ffn), m, what) == (B.FORM_GEMM, *route)


def test_layer_routes_refuse_what_is_no_gemm_of_a_layer():
    c = layer_config(100, 128, 512)
    for n_rows, what in ((0, B.ROUTE_QKV), (101, B.ROUTE_QKV), (100, B.ROUTE_GELU), (100, B.ROUTE_FFN2 + 1)):
        with pytest.raises(B.HeroError):
            B.hero_layer_route(c, n_rows, what)
    with pytest.raises(B.HeroError):
        B.hero_layer_route(layer_config(100, 128, 100), 100, B.ROUTE_QKV)


@pytest.mark.parametrize("r,n_keys,heads,queries", [
    (326, 33976, 40, 256),       # 168 us against 217
    (1306, 33976, 12, 256),      # 157 against 174
    (1000, 8218, 30, 256),       # 73 against 76
    (326, 326, 4, 32),           # 7.8 (64 queries) against 15
    (500, 2000, 4, 32),          # 10.0 us; 64 queries 13.3
    (1000, 2000, 8, 32),         # 10.7; 13.9
    (691, 2032, 16, 64),         # 14.8; 32 queries 16.0
    (2032, 2032, 16, 64),        # 25 against 37
    (4485, 17776, 48, 256),
])
def test_measured_attention_choices(r, n_keys, heads, queries):
    assert B.hero_attention_route(r, n_keys, heads, 64, 128 * MIB)[0] == queries


def kernels(c, rows, listed):
    """The kernels of a layer's four GEMMs: which GEMM, on listed rows or not, form, tile, and whether the tiles are cut (the
    narrow models' kernel: how many workgroups share)."""
    for what in (B.ROUTE_QKV, B.ROUTE_OUT, B.ROUTE_FFN1, B.ROUTE_FFN2):
        form, tm, tn, chunks = B.hero_layer_route(c, rows, what, listed)
        yield what, listed, form, tm, tn, chunks if form == B.FORM_TAIL else chunks > 1


def test_the_blocks_that_the_gpu_tests_run_take_every_kernel():
    configs = [block_config(*shape) for shape in BLOCKS]
    configs += [test_gpu_gemm_cut.config(*shape) for shape in test_gpu_gemm_cut.SHAPES]
    configs += [test_gpu_narrow.config(s[0], widths * 64 * s[0], *s[1:]) for s in test_gpu_narrow.NORMALISING for widths in (3, 4)]
    configs += [test_gpu_narrow.config(s[0], 256 * s[0], *s[1:5]) for s in test_gpu_narrow.ONE_KERNEL]
    run = set()
    for cfg in configs:
        c = B.make_config(cfg)
        run.update(kernels(c, cfg.n_tokens, False))
        run.update(kernels(c, B.hero_num_selected(c), True))
    reachable, rng = set(), random.Random(1)
    for heads in (*range(1, 49), 52, 64, 96, 128):
        for ffn in (64, 320, 1088, 64 * heads, 128 * heads, 256 * heads, 9216):
            for _ in range(24):
                tokens = int(2 ** rng.uniform(0, 14.7))
                if (tokens + 512) * max(64 * heads, ffn) * 2 >= 2 ** 32:
                    continue
                c = layer_config(tokens, 64 * heads, ffn)
                reachable.update(kernels(c, tokens, False))
                reachable.update(kernels(c, max(1, int(tokens * rng.choice((0.5, 0.25, 0.1)))), True))
    assert len(reachable) > 80
    assert reachable <= run, sorted(reachable - run)
