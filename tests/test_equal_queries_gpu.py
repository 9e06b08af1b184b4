"""Queries with the same row and the same samples have the same measure to the last bit wherever they lie, on every route
of the measure stage.  Ties go to the lower index, so rounding must not tell such queries apart."""
import numpy as np
import pytest

from paper_2106_09236_amd import workloads as W
from tests.test_parity_gpu import gpu_forward
from tests.test_plan import plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,B,H,L,U,measure,parts", [
    ("f32", 16, 4, 750, 34, "stream", 2), ("f32", 16, 4, 1000, 38, "stream", 2),
    ("bf16", 5, 8, 1200, 35, "stream", 2), ("bf16", 8, 8, 2048, 39, "stream", 4),
    ("f32", 2, 4, 800, 24, "stream", 0), ("bf16", 2, 4, 1500, 24, "stream", 0), ("f32", 2, 4, 600, 70, "stream", 0), ("bf16", 2, 4, 1200, 70, "stream", 0),
    # heads in LDS: chunks of 32, 64 and 128 queries, of two quads and of one to a query
    ("f32", 2, 4, 128, 25, "lds", 0), ("f32", 2, 4, 333, 30, "lds", 0), ("f32", 20, 8, 250, 28, "lds", 0), ("f32", 16, 4, 512, 32, "lds", 0),
    ("bf16", 2, 4, 128, 25, "lds_half", 0), ("bf16", 2, 4, 333, 30, "lds_half", 0), ("bf16", 32, 4, 512, 32, "lds_half", 0), ("bf16", 16, 8, 1000, 35, "lds", 0),
    ("f32", 16, 4, 500, 56, "lds", 0), ("bf16", 32, 4, 512, 56, "lds_half", 0),
])
def test_same_bits(dtype, B, H, L, U, measure, parts):
    p = plan(B, H, L, U, dtype)
    assert (p["measure"], int(p["measure_parts"])) == (measure, parts)
    w = W.make_workload(W.small_config("equal", B, H, L, U, 5.0, dtype, "normal", True, L // 2, L), seed=L + U)
    w.lengths[:2] = L, L - 37                              # whole chunks and one that is cut
    rng = np.random.default_rng(U)
    source = {}
    for b in range(2):
        n = int(w.lengths[b])
        for h in range(H):
            # each of the last two thirds of the rows is like one of the first third
            source[b, h] = src = np.concatenate([np.arange(n // 3), rng.integers(0, n // 3, size=n - n // 3)])
            for x in (w.Q, w.K, w.V):                      # (the item may be longer than it was drawn)
                x[b, h, :n] = x[b, h, rng.integers(0, L // 2, size=n)]
            w.sample_idx[b, h, :n] = rng.integers(0, n, size=(n, U))
            w.Q[b, h, :n], w.sample_idx[b, h, :n] = w.Q[b, h, src], w.sample_idx[b, h, src]
    _, M, sel, u = gpu_forward(w)
    for (b, h), src in source.items():
        n = len(src)
        assert (M[b, h, :n] == M[b, h, src]).all(), (b, h, np.flatnonzero(M[b, h, :n] != M[b, h, src]))
        kept = np.zeros(n, dtype=bool)
        kept[sel[b, h, :int(u[b])]] = True
        for i in np.flatnonzero(kept):                     # the lower ones first
            assert kept[:i][src[:i] == src[i]].all(), (b, h, i)
