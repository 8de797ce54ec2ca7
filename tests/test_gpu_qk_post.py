"""q / k post-processing at the widths where a wave's walk over a row ends differently: part of one
512-channel pass, a pass and a remainder, a batch of three passes and a remainder.  The keys of a block
with head LayerNorm and rotation, against the same block's keys without, post-processed in float64."""
import numpy as np
import pytest
import torch

from oracle import hero_oracle as O
from paper_2508_17588_amd import binding as B
from workloads import BLOCK_QKNORM, BLOCK_ROPE, get_config
from hero_testlib import to_host_f64
from torch_block import weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,head_dim", [(1, 64), (6, 32), (9, 64), (24, 64), (25, 64), (50, 32)])
@pytest.mark.parametrize("flags", [BLOCK_QKNORM, BLOCK_ROPE, BLOCK_QKNORM | BLOCK_ROPE])
def test_keys_are_the_plain_keys_post_processed(heads, head_dim, flags):
    d = heads * head_dim
    print(f"[case] hidden {d}, head_dim {head_dim}, flags {flags}", flush=True)
    base = dict(n_layers=1, n_shallow=1, hidden=d, n_heads=heads, head_dim=head_dim, ffn_dim=4 * d, frames=2, height=5,
                width=7, n_text=3)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    plain, post = get_config("tiny", block_flags=0, **base), get_config("tiny", block_flags=flags, **base)
    w = weights(plain, gen, most=1600)
    if flags & BLOCK_QKNORM:
        for n in ("q_norm", "k_norm"):
            w[n + "_g"] = (torch.randn(head_dim, generator=gen, device="cuda") * 0.1 + 1).to(torch.bfloat16)
            w[n + "_b"] = (torch.randn(head_dim, generator=gen, device="cuda") * 0.1).to(torch.bfloat16)
    caches = [B.HeroCache(B.make_config(c)) for c in (plain, post)]
    names = set(weights(plain, gen, most=1600))
    caches[0].hero_set_layer_weights(0, {n: t for n, t in w.items() if n in names})
    caches[1].hero_set_layer_weights(0, w)
    n, idx = plain.n_tokens, torch.zeros(plain.n_tokens, dtype=torch.int32, device="cuda")
    for call in ("full", "refresh"):
        x = torch.randn(n, d, generator=gen, device="cuda")
        keys = []
        for c in caches:
            if call == "full":
                c.hero_full_layer(0, x.clone())
            else:
                n_sel = c.hero_select(1, idx)
                c.hero_refresh_layer(0, x.clone(), idx, n_sel)
            torch.cuda.synchronize()
            keys.append(to_host_f64(c.hero_cache_view(0, B.VIEW_K)))
        want = keys[0]
        if flags & BLOCK_QKNORM:
            want = O.head_layer_norm(want, to_host_f64(w["k_norm_g"]), to_host_f64(w["k_norm_b"]), heads)
        if flags & BLOCK_ROPE:
            want = want.copy()
            want[3:] = O.apply_rope(want[3:], O.rope_angles(2, 5, 7, head_dim), heads)
        # one rounding to bf16, and fp32 arithmetic on values of up to some 8 in between
        err = np.abs(keys[1] - want)
        assert (err <= 2.0 ** -8 * np.abs(want) + 2e-5).all(), f"{call}: off by {err.max()}"
    for c in caches:
        c.close()
