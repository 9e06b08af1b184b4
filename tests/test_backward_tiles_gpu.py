"""The backward at the edges of its tiles: query tiles of 16, groups of 32 and 64, key blocks of 32 and 64, several
key blocks per work-group, and more kept queries than the gradient kernel keeps statistics of (768)."""
import numpy as np
import pytest
import torch

from paper_2106_09236_amd import workloads as W
from tests.test_backward_gpu import check_backward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,H,L,u", [
    (1, 2, 63, 16), (1, 2, 64, 17), (1, 1, 129, 33), (2, 2, 1000, 65),   # few heads: blocks of 32 keys
    (40, 4, 130, 32), (64, 8, 65, 31), (8, 8, 700, 64),                  # many: blocks of 64, several per work-group
    (1, 1, 1700, 768), (1, 1, 1700, 769),                                # statistics in LDS, and put together anew
])
def test_tiles(dtype, B, H, L, u):
    cfg = W.small_config("t", B, H, L, 4, 5.0, dtype, "mixture", B > 1, max(1, L // 2), L)
    w = W.make_workload(cfg, seed=900 + L + u)
    r = np.random.Generator(np.random.PCG64(L + u))
    n = w.lengths_or_full()
    sel = np.full((B, H, u), -1, dtype=np.int32)
    ub = np.minimum(u, n).astype(np.int32)
    for b in range(B):
        for h in range(H):
            sel[b, h, :ub[b]] = r.permutation(int(n[b]))[:ub[b]]
    check_backward(w, torch.from_numpy(sel).cuda(), torch.from_numpy(ub).cuda(), "mean" if u % 2 else "value",
                   label=f"tiles B{B} H{H} L{L} u{u} {dtype}")
