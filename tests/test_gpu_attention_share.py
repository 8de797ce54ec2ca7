"""Attention with few query blocks (32 or 64 queries a workgroup, its waves share the keys): key counts around a
tile and around what gives every wave one, ragged query counts, and the count of blocks that leave the
reference-free form."""
import numpy as np
import pytest
import torch

from oracle import hero_oracle as O
from paper_2508_17588_amd import binding as B
from workloads import round_to_bf16
from hero_testlib import assert_close, to_dev_bf16, to_host_f64

pytestmark = pytest.mark.gpu


def rnd(seed, *shape):
    return round_to_bf16(np.random.default_rng(seed).standard_normal(shape, dtype=np.float32))


def run(r, n_keys, heads, hd, bad_queries=()):
    print(f"[case] attention r={r} n_keys={n_keys} heads={heads} hd={hd} bad={bad_queries}", flush=True)
    d, ld = heads * hd, (n_keys + 63) // 64 * 64
    q, k, v = rnd(1, r, d), rnd(2, n_keys, d), rnd(3, n_keys, d)
    for i in bad_queries:
        q[i] = round_to_bf16(q[i] * 200)
    vt = np.zeros((d, ld), np.float32)
    vt[:, :n_keys] = v.T
    o = torch.full((r + 1, d), 3.0, dtype=torch.bfloat16, device="cuda")
    count = torch.zeros(1, dtype=torch.int32, device="cuda")
    B.hero_attention(to_dev_bf16(q), to_dev_bf16(k), to_dev_bf16(vt), o, n_keys, heads, hd, None, count)
    torch.cuda.synchronize()
    assert_close(to_host_f64(o[:r]), O.attention(q.astype(np.float64), k.astype(np.float64), v.astype(np.float64), heads), "attention")
    assert float((o[r:] - 3.0).abs().max()) == 0.0
    return int(count.item())


@pytest.mark.parametrize("hd", [32, 64])
@pytest.mark.parametrize("r,n_keys,heads", [(1, 1, 1), (63, 63, 3), (64, 64, 2), (65, 65, 3), (129, 192, 2), (200, 255, 3),
                                            (256, 257, 2), (321, 513, 5), (700, 2033, 4)])
def test_key_and_query_counts(r, n_keys, heads, hd):
    assert B.hero_attention_route(r, n_keys, heads, hd) == (32, 1)
    assert run(r, n_keys, heads, hd) == 0


@pytest.mark.parametrize("bad,blocks", [((77,), 1), ((3, 77, 130, 255), 1), ((255,), 1), ((70, 290), 2), ((256, 299), 1)])
def test_a_block_of_256_queries_is_counted_once(bad, blocks):
    assert B.hero_attention_route(300, 700, 3, 64) == B.hero_attention_route(300, 700, 3, 32) == (32, 1)
    assert run(300, 700, 3, 64, bad) == 3 * blocks
    assert run(300, 700, 3, 32, bad) == 0            # only head_dim 64 keeps a count


# more than 256 blocks of 32 queries: 64 to a workgroup; up to 256: 32
@pytest.mark.parametrize("hd", [32, 64])
@pytest.mark.parametrize("r,n_keys,heads,queries", [(1, 65, 256, 32), (1, 65, 257, 64), (33, 63, 128, 32), (33, 64, 129, 64),
                                                    (65, 65, 90, 64), (200, 255, 40, 64), (256, 257, 32, 32), (257, 257, 32, 64),
                                                    (300, 513, 27, 64)])
def test_either_number_of_queries_to_a_workgroup(r, n_keys, heads, queries, hd):
    assert B.hero_attention_route(r, n_keys, heads, hd) == (queries, 1)
    assert run(r, n_keys, heads, hd) == 0


@pytest.mark.parametrize("bad,blocks", [((77,), 1), ((3, 77, 130, 255), 1), ((70, 290), 2), ((256, 299), 1)])
def test_a_block_is_counted_once_with_64_queries_to_a_workgroup(bad, blocks):
    assert B.hero_attention_route(300, 700, 27, 64) == B.hero_attention_route(300, 700, 27, 32) == (64, 1)
    assert run(300, 700, 27, 64, bad) == 27 * blocks
    assert run(300, 700, 27, 32, bad) == 0
