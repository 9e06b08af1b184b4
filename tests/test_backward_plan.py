"""Scratch memory of the backward (host arithmetic, no GPU): the partial sums of dQ stay within what the header says."""
import ctypes
import random

import pytest

from paper_2106_09236_amd import binding as psa


def scratch(B, H, L, u, dtype):
    shape = psa.make_shape(B, H, L, 1, psa.PSA_F32 if dtype == "f32" else psa.PSA_BF16)
    return psa.load().probsparse_attn_bwd_workspace_bytes(ctypes.byref(shape), u)


def bound(B, H, L, u, dtype):
    tensors = 7 * B * H * L * 64 * (4 if dtype == "f32" else 2)
    # statistics (24 bytes per query and key split, 16 per query), column sums of dOut (512 bytes per head and split): with
    # few work-groups the keys are split, which stays below 16 MB
    return max(256 << 20, tensors // 4) + B * H * (40 * (u + 16) + 1024) + (16 << 20)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,H,L,u,most", [
    (16, 4, 512, 256, 70), (24, 4, 750, 375, 155), (8, 8, 2048, 1024, 275), (1, 8, 16384, 8192, 4), (222, 16, 53875, 53800, 7800),
    (1, 4, 2000, 1000, 2), (8, 8, 2048, 39, 14),
])
def test_known_shapes(B, H, L, u, most, dtype):
    assert 0 < scratch(B, H, L, u, dtype) <= min(most * 10 ** 6, bound(B, H, L, u, dtype))


def test_bound_holds_over_the_range():
    rng = random.Random(3)
    for _ in range(4000):
        B, H, L = int(2 ** rng.uniform(0, 9)), rng.choice([1, 4, 8, 16]), int(2 ** rng.uniform(0, 17))
        u = max(1, min(L, int(L * 2 ** rng.uniform(-9, 0))))
        dtype = rng.choice(["f32", "bf16"])
        assert 0 < scratch(B, H, L, u, dtype) <= bound(B, H, L, u, dtype), (B, H, L, u, dtype)
