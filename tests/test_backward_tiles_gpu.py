"""The backward at the edges of its tiles: query tiles of 16, groups of 32 and 64, key blocks of 32 and 64, several
key blocks per work-group, more kept queries than the gradient kernel keeps statistics of (768), and dQ from a kernel
of its own (no partial sums, which the scratch size shows)."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2106_09236_amd import binding as psa
from paper_2106_09236_amd import workloads as W
from tests.test_backward_gpu import check_backward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,H,L,u", [
    (1, 2, 63, 16), (1, 2, 64, 17), (1, 1, 129, 33), (2, 2, 1000, 65),   # few heads: blocks of 32 keys
    (40, 4, 130, 32), (64, 8, 65, 31), (8, 8, 700, 64),                  # many: blocks of 64, several per work-group
    (1, 1, 1700, 768), (1, 1, 1700, 769),                                # the most statistics kept in LDS, one more
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


def _scratch(B, H, L, u, dtype):
    shape = psa.make_shape(B, H, L, 1, psa.PSA_F32 if dtype == "f32" else psa.PSA_BF16)
    return psa.load().probsparse_attn_bwd_workspace_bytes(ctypes.byref(shape), u)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,H,L,u,partial_sums", [
    (16, 4, 900, 800, True), (9, 8, 830, 830, True),                     # statistics put together anew for every block
    (1, 1, 770, 769, False), (3, 2, 1000, 900, False), (1, 2, 2047, 785, False), (2, 3, 1025, 1025, False),
    (1, 8, 4096, 2048, False),                                           # blocks of 64 keys: the partial sums are bounded
])
def test_many_kept_queries(dtype, B, H, L, u, partial_sums):
    u_pad = (u + 15) // 16 * 16
    assert (_scratch(B, H, L, u, dtype) >= B * H * 2 * u_pad * 512) == partial_sums
    test_tiles(dtype, B, H, L, u)
