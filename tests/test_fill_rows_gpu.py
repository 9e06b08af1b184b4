"""Rows that the attend work-groups fill: shares that end at, before and behind 4, 8 and 16 stores per thread (32 rows each for float32, 64
for bfloat16) and behind a block of 512 flags, with selected rows at both ends of a share, for every way the selection reaches
the work-groups."""
import numpy as np
import pytest

from paper_2106_09236_amd import workloads as W
from tests.test_parity_gpu import check_against_oracle
from tests.test_plan import plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ragged", [False, True])
@pytest.mark.parametrize("dtype,B,H,L,select,rows", [
    ("f32", 8, 8, 512, "lists", 128), ("f32", 24, 4, 129, "lists", 65), ("f32", 40, 4, 256, "lists", 256), ("f32", 40, 4, 257, "lists", 257),
    ("f32", 70, 4, 512, "lists", 512), ("f32", 70, 2, 513, "lists", 513), ("f32", 1, 8, 16384, "segments", 512), ("f32", 8, 8, 2048, "lists", 683),
    ("bf16", 24, 4, 129, "lists", 129), ("bf16", 40, 4, 256, "lists", 256), ("bf16", 40, 4, 257, "lists", 257), ("bf16", 70, 4, 512, "lists", 512),
    ("bf16", 70, 4, 513, "lists", 513), ("bf16", 8, 8, 2048, "lists", 512), ("bf16", 4, 8, 2048, "kernel", 256),
])
def test_shares(dtype, B, H, L, select, rows, ragged):
    p = plan(B, H, L, 8, dtype)
    shares = int(p["key_splits"]) * int(p["query_groups"]) * int(p["element_shares"])
    assert p["attend"] == "key_split" and p["select"] == select
    if (dtype, L) != ("f32", 513):                                   # (there the cut may be another)
        assert -(-L // shares) == rows
    w = W.make_workload(W.small_config("fill", B, H, L, 8, 5.0, dtype, "normal", ragged, max(1, L // 3), L), seed=60 + L)
    # the kept queries lie at the ends of the shares and of blocks of 512 flags
    for first in range(0, L, rows):
        for i in (first, min(L, first + rows) - 1, min(L - 1, first + 511)):
            w.Q[:, :, i] = w.Q[:, :, i] * 8 if w.Q.dtype != np.uint16 else w.Q[:, :, (i + 1) % L]
    for b in range(B):
        w.Q[b, :, int(w.lengths_or_full()[b]):] = 0
    check_against_oracle(w, label=f"fill {dtype} B{B} H{H} L{L} ragged={ragged}")
