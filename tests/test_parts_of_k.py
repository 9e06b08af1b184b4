"""The measure of streamed heads whose K goes through LDS in two parts: which calls take it, and the edges of its passes
(128 queries), lists (256) and copies of K (192 and 256 KB), sample counts on both sides of a round of 4 and of what it takes
(29 to 40), heads in eights and not."""
import numpy as np
import pytest

from paper_2106_09236_amd import workloads as W
from tests.test_parity_gpu import check_against_oracle, gpu_forward
from tests.test_plan import plan


@pytest.mark.parametrize("dtype,B,H,L,U,passes", [
    ("f32", 16, 4, 750, 34, 2), ("f32", 16, 4, 1024, 35, 2), ("f32", 22, 4, 513, 32, 2), ("bf16", 8, 8, 2048, 39, 4),
    ("bf16", 3, 8, 2048, 39, 2), ("bf16", 5, 8, 1040, 35, 2), ("bf16", 12, 8, 1040, 35, 4), ("bf16", 7, 4, 1281, 29, 2), ("bf16", 20, 8, 1200, 36, 4),
    # bfloat16: a round that is not full, with few samples; one round of few work-groups, of few heads
    ("bf16", 8, 8, 1300, 36, 0), ("bf16", 9, 8, 2048, 39, 0), ("bf16", 12, 8, 2048, 39, 0), ("bf16", 14, 8, 1400, 37, 0), ("bf16", 8, 8, 2048, 29, 0),
    ("bf16", 16, 4, 2000, 31, 4), ("bf16", 7, 4, 1100, 36, 0), ("bf16", 3, 8, 1600, 37, 0),
    # heads that fit LDS whole, or not in two parts; few and many samples; few work-groups
    ("f32", 22, 4, 512, 32, 0), ("f32", 16, 4, 1025, 35, 0), ("bf16", 32, 8, 1024, 35, 0), ("bf16", 8, 8, 2049, 39, 0),
    ("f32", 16, 4, 750, 28, 0), ("f32", 16, 4, 750, 29, 2), ("f32", 16, 4, 750, 40, 2), ("f32", 16, 4, 750, 41, 0),
    ("f32", 8, 4, 1024, 35, 0), ("f32", 11, 4, 750, 34, 2), ("bf16", 2, 8, 2048, 39, 0),
])
def test_calls_that_take_it(dtype, B, H, L, U, passes):
    p = plan(B, H, L, U, dtype)
    assert int(p["measure_parts"]) == passes
    if passes:
        assert (p["measure"], p["select"], int(p["lists"])) == ("stream", "lists", -(-L // 256))
        assert int(p["chunks_per_wg"]) == 2 * passes                 # of the kernel that is launched
        # half of the queries kept: the same measure, and the select kernel
        r = plan(B, H, L, U, dtype, r_sparse=0.5)
        assert (int(r["measure_parts"]), r["select"]) == (passes, "kernel")


def _workload(dtype, B, H, L, U, ragged):
    w = W.make_workload(W.small_config("parts", B, H, L, U, 5.0, dtype, "peaky", ragged, 1, L), seed=300 + L + U)
    if ragged:
        for b, n in enumerate([L, 0, 1, 127, 128, 129, 256, 257, L - 1]):
            if b < B and n <= L:
                w.lengths[b] = n
                w.sample_idx[b] = np.minimum(w.sample_idx[b], max(0, n - 1))
        for b in range(B):
            for x in (w.Q, w.K, w.V):
                x[b, :, int(w.lengths[b]):] = 0
    return w


@pytest.mark.gpu
@pytest.mark.parametrize("ragged", [False, True])
@pytest.mark.parametrize("dtype,B,H,L,U", [
    ("f32", 15, 3, 513, 29), ("f32", 43, 1, 768, 36), ("f32", 9, 4, 769, 37), ("f32", 33, 1, 1023, 40), ("f32", 11, 3, 1024, 33),
    ("bf16", 33, 1, 1025, 40), ("bf16", 14, 2, 1536, 36), ("bf16", 29, 1, 1537, 29), ("bf16", 25, 1, 2047, 37), ("bf16", 5, 5, 2048, 33),
    ("bf16", 25, 2, 2048, 39), ("bf16", 126, 1, 1281, 40), ("bf16", 61, 2, 1040, 39),      # four passes
])
def test_edges(dtype, B, H, L, U, ragged):
    assert int(plan(B, H, L, U, dtype)["measure_parts"]) in (2, 4)
    check_against_oracle(_workload(dtype, B, H, L, U, ragged), label=f"parts {dtype} B{B} H{H} L{L} U{U} ragged={ragged}")


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,B,H,L,U", [("f32", 12, 4, 700, 35), ("bf16", 4, 8, 1300, 39), ("bf16", 12, 4, 2048, 40)])
def test_ties_samples_out_of_range_and_padding(dtype, B, H, L, U):
    """Equal measures across the chunks of a list and across lists, a head of equal measures, unusable samples, NaN behind the lengths."""
    assert int(plan(B, H, L, U, dtype)["measure_parts"]) in (2, 4)
    w = _workload(dtype, B, H, L, U, True)
    w.lengths[2] = L
    w.sample_idx[2] = np.random.default_rng(5).integers(0, L, size=w.sample_idx[2].shape)
    w.Q[2, 0] = 0                                                                          # all equal
    for first in (64, 192, 256, 448, 512):
        m = min(64, L - first)
        w.Q[2, 1, first:first + m] = w.Q[2, 1, :m]
        w.sample_idx[2, 1, first:first + m] = w.sample_idx[2, 1, :m]
    w.sample_idx[0, :, 5::7, 3] = -1
    w.sample_idx[0, :, 6::11, :] = L
    w.sample_idx[0, 0, 130, 1:] = 1 << 30
    for b in range(B):
        for x in (w.Q, w.K, w.V):
            x[b, :, int(w.lengths[b]):] = np.nan if x.dtype != np.uint16 else 0x7FC0
    check_against_oracle(w, label=f"parts ties {dtype} L{L}")
    u2 = int(gpu_forward(w)[3][2])
    assert sorted(gpu_forward(w)[2][2, 0, :u2].tolist()) == list(range(u2))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,B,H,L,U", [("f32", 15, 3, 515, 34), ("bf16", 4, 9, 1100, 35), ("bf16", 32, 4, 1281, 39)])
def test_without_lists(dtype, B, H, L, U):
    # half of the queries kept: column sums per chunk and the measures themselves go to the select kernel
    p = plan(B, H, L, U, dtype, r_sparse=0.5)
    assert int(p["measure_parts"]) in (2, 4) and p["select"] == "kernel"
    check_against_oracle(_workload(dtype, B, H, L, U, True), r_sparse=0.5, fill="mean", label=f"parts select {dtype} L{L}")
