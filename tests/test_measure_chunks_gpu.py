"""The measure of short heads in chunks of 32, 64 and 128 queries: chunk edges, sample counts around a round of 8 and
around what is fetched up front (40), ragged lengths."""
import pytest

from paper_2106_09236_amd import workloads as W
from tests.test_parity_gpu import check_against_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,H,L,U", [
    (1, 4, 32, 1), (2, 4, 33, 7), (3, 2, 65, 8), (1, 4, 128, 25), (2, 2, 255, 9), (1, 8, 256, 41),     # chunks of 32
    (1, 4, 257, 3), (2, 4, 320, 40), (1, 4, 512, 48), (3, 8, 500, 31),                                # chunks of 64
    (40, 8, 65, 12), (80, 8, 129, 5), (9, 4, 511, 25),                                                # chunks of 128, many heads
])
def test_chunks(dtype, B, H, L, U):
    cfg = W.small_config("chunks", B, H, L, U, 3.0, dtype, "mixture", B > 1, max(1, L // 3), L)
    check_against_oracle(W.make_workload(cfg, seed=500 + L + U), label=f"B{B} H{H} L{L} U{U} {dtype}")
