"""Selection over patches around the sizes that are held in registers (4, 8 and 16 tokens) and past them, clipped at the
grid's edges, both readings, bit for bit against the oracle."""
import numpy as np
import pytest
import torch

from oracle import hero_oracle as O
from paper_2508_17588_amd import binding as B
from workloads import get_config

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("patch_h,patch_w", [(1, 1), (2, 2), (1, 5), (2, 4), (3, 3), (3, 5), (4, 4), (1, 17), (4, 5), (9, 14)])
@pytest.mark.parametrize("ratio", [0.1, 0.5, 1.0])
def test_patches_of_every_size(patch_h, patch_w, ratio, mode):
    cfg = get_config("tiny", n_layers=1, n_shallow=1, hidden=64, n_heads=1, head_dim=64, ffn_dim=64, frames=2, height=9,
                     width=14, n_text=3, patch_h=patch_h, patch_w=patch_w, ratio=ratio, select_mode=mode)
    cache = B.HeroCache(B.make_config(cfg))
    n_sel = B.hero_num_selected(cache.cfg)
    idx = torch.full((n_sel,), -1, dtype=torch.int32, device="cuda")
    ages = np.zeros(cfg.n_video, np.int32)
    for step in (1, 2, 3, 5, 1000003):
        want, ages = O.select(ages, cfg, step)
        assert cache.hero_select(step, idx) == n_sel == len(want)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(idx.cpu().numpy(), want)
        np.testing.assert_array_equal(cache.hero_cache_view(0, B.VIEW_AGES).cpu().numpy(), ages)
    cache.close()
