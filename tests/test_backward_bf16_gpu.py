"""The backward of bfloat16 tensors at the edges of its tiles (32 kept queries, 64 staged, 32 keys, blocks of 128, 2048 rows to a
bit mask) and where its float32 arithmetic could go wrong: attention on one key, scores far below zero beside a ragged
tail, keys with much in common.  Against the float64 oracle at the tolerance of tests/test_backward_gpu.py."""
import numpy as np
import pytest
import torch

from paper_2106_09236_amd import workloads as W
from tests.test_backward_gpu import check_backward

pytestmark = pytest.mark.gpu


def _workload(B, H, L, ragged, values="mixture", seed=1):
    return W.make_workload(W.small_config("b16", B, H, L, 4, 5.0, "bf16", values, ragged, max(1, L // 2), L), seed=seed)


def _sets(w, u, seed):
    """Random sets of up to u distinct valid queries; every seventh entry absent."""
    r = np.random.Generator(np.random.PCG64(seed))
    n, cfg = w.lengths_or_full(), w.cfg
    ub = np.minimum(u, n).astype(np.int32)
    sel = np.full((cfg.B, cfg.H, u), -1, dtype=np.int32)
    for b in range(cfg.B):
        for h in range(cfg.H):
            sel[b, h, :ub[b]] = r.permutation(int(n[b]))[:ub[b]]
            sel[b, h, 6:ub[b]:7] = -1
    return torch.from_numpy(sel).cuda(), torch.from_numpy(ub).cuda()


@pytest.mark.parametrize("fill", ["mean", "value"])
@pytest.mark.parametrize("B,H,L,u", [
    (1, 1, 1, 1), (1, 2, 32, 32), (2, 1, 33, 31), (1, 3, 127, 33), (2, 4, 128, 16), (1, 8, 129, 17),
    (2, 8, 257, 65), (1, 2, 2049, 129),           # a second bit mask, column sums dealt to three groups of queries
    (1, 1, 3000, 40), (2, 4, 1500, 64),           # keys split for the statistics and for dQ
    (64, 8, 150, 30), (40, 8, 600, 70),           # several blocks of keys to a work-group, with one group of queries and with two
])
def test_tiles(B, H, L, u, fill):
    w = _workload(B, H, L, B > 1, seed=300 + L + u)
    check_backward(w, *_sets(w, u, L + u), fill, label=f"B{B} H{H} L{L} u{u} {fill}")


def _bf16(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)


@pytest.mark.parametrize("L,u", [(61, 20), (700, 48), (1500, 300)])
def test_attention_on_one_key(L, u):
    # a kept query is four times a key: its heaviest key holds all but 1e-5 .. 1e-12 of the weight, and the gradients of Q and K are
    # as small (every kept query's, so that nothing larger hides them in the tolerance's floor)
    w = _workload(1, 2, L, False, "normal", seed=L)
    sel, ub = _sets(w, u, L)
    Q, K = w.as_f64("Q").copy(), w.as_f64("K")
    for h in range(2):
        for i in sel[0, h].cpu().numpy():
            if i >= 0:
                Q[0, h, i] = 4.0 * K[0, h, (7 * i) % L]
    w.Q[...] = _bf16(Q)
    check_backward(w, sel, ub, "value", label=f"one key L{L}")


@pytest.mark.parametrize("sign", [-1.0, 1.0])
def test_scores_far_from_zero(sign):
    # all scores near -200 or +200: a masked key's zero must not count as a score, and what the keys have in common (sixteen times
    # their spread) must not enter dQ, which a float32 sum over 3 rows in common with errors of 1e-7 would show
    w = _workload(3, 2, 77, True, "normal", seed=8)
    sel, ub = _sets(w, 20, 8)
    w.K[...] = _bf16(5.0 + 0.3 * w.as_f64("K"))
    w.Q[...] = _bf16(sign * 5.0 + 0.3 * w.as_f64("Q"))
    check_backward(w, sel, ub, "mean", label=f"far {sign}")
