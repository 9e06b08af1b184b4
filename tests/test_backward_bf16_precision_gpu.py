"""Precision of the backward of bfloat16 tensors: the error (2-norm) of each gradient against the float64 oracle is that of rounding the
oracle's own result to bfloat16, with 1 % on top, which leaves the arithmetic before the rounding a seventh of the rounding's error
(both are independent: sqrt(1 + 0.14^2) = 1.01).  Over the shapes and values of ordinary calls, and for heads whose values float32
would not carry: large scores, rows with much in common beside their differences, extreme scales, infinite gradients."""
import numpy as np
import pytest
import torch

from oracle import probsparse_oracle as O
from paper_2106_09236_amd import binding as psa
from paper_2106_09236_amd import workloads as W
from tests.test_backward_bf16_gpu import _bf16, _sets, _workload

pytestmark = pytest.mark.gpu


def _gradients(w, sel, u, G, fill):
    def dev(a):
        return torch.from_numpy(a.view(np.int16)).view(torch.bfloat16).cuda()
    lengths = None if w.lengths is None else torch.from_numpy(w.lengths).cuda()
    got = psa.probsparse_attn_bwd(dev(w.Q), dev(w.K), dev(w.V), lengths, sel, u, dev(G), psa.FILL_VALUE if fill == "value" else psa.FILL_MEAN)
    sel_h, n = sel.cpu().numpy(), w.lengths_or_full()
    sets = [[np.array([i for i in row[:int(u[b])] if 0 <= i < int(n[b])], dtype=np.int64) for row in sel_h[b]] for b in range(w.cfg.B)]
    with np.errstate(invalid="ignore", over="ignore"):
        ref = O.attention_with_indices_backward(w.as_f64("Q"), w.as_f64("K"), w.as_f64("V"), w.lengths, sets, W.to_f64(G, "bf16"), fill=fill)
    return [x.float().cpu().numpy().astype(np.float64) for x in got], ref, sets


def _check(got, ref, label, heads=None):
    for name, g, r in zip(("dQ", "dK", "dV"), got, ref):
        if heads is not None:
            g, r = g[:, heads], r[:, heads]
        size = max(np.linalg.norm(r), 1e-300)
        err, rounding = np.linalg.norm(g - r), np.linalg.norm(O.round_to(r, "bf16") - r)
        print(label, name, err / size, rounding / size, flush=True)
        assert err <= 1.01 * rounding, f"{label}: {name} off by {err / size:.3e}, the rounding alone by {rounding / size:.3e}"


@pytest.mark.parametrize("values", ["normal", "peaky", "mixture"])
@pytest.mark.parametrize("B,H,L,u,ragged", [
    (6, 8, 40, 19, False), (4, 4, 128, 25, False), (5, 4, 333, 30, True), (1, 8, 2048, 39, False),
    (2, 4, 700, 350, True), (1, 2, 16384, 49, False), (1, 1, 3001, 1500, False),
])
def test_error_is_that_of_the_last_rounding(B, H, L, u, ragged, values):
    w = _workload(B, H, L, ragged, values, seed=60 + L)
    sel, ub = _sets(w, u, L)
    fill = "value" if u % 2 else "mean"
    got, ref, _ = _gradients(w, sel, ub, W.make_upstream_gradient(w.cfg, 5, lengths=w.lengths), fill)
    _check(got, ref, f"{values} B{B} H{H} L{L} u{u}")


def _large_scores(Q, K, V, G):
    # half of the elements in common, 80 * 300 a product: scores of 96000 and differences of a few units between them
    Q[..., :32], K[..., :32] = 80.0, 300.0


def _offset_values(Q, K, V, G):
    V[..., :32] = 30000.0


def _offset_keys(Q, K, V, G):
    Q[..., :32], K[..., :32] = 0.0, 30000.0


def _scaled(Q, K, V, G):
    Q *= 2.0 ** 60
    K *= 2.0 ** -60
    V *= 2.0 ** -50
    G *= 2.0 ** -40


def _within(Q, K, V, G):
    # scores of 800, values with 100 times their differences in common: what float32 carries still
    Q[..., :32], K[..., :32] = 10.0, 15.0
    V[..., :32] = 150.0


def _within_keys(Q, K, V, G):
    Q[..., :32], K[..., :32] = 0.0, 80.0


HARD = {"large scores": _large_scores, "offset values": _offset_values, "offset keys": _offset_keys, "scaled": _scaled,
        "within": _within, "keys within": _within_keys}


def _one_hard_head(kind, B, H, L, u, ragged, seed):
    w = _workload(B, H, L, ragged, "normal", seed=seed)
    sel, ub = _sets(w, u, seed)
    G = W.make_upstream_gradient(w.cfg, 5, lengths=w.lengths)
    a = {k: w.as_f64(k).copy() for k in "QKV"}
    g = W.to_f64(G, "bf16").copy()
    HARD[kind](a["Q"][:, 1], a["K"][:, 1], a["V"][:, 1], g[:, 1])
    w.Q[...], w.K[...], w.V[...] = _bf16(a["Q"]), _bf16(a["K"]), _bf16(a["V"])
    return w, sel, ub, _bf16(g)


@pytest.mark.parametrize("kind", sorted(HARD))
@pytest.mark.parametrize("B,H,L,u,ragged", [
    (8, 2, 60, 25, False), (2, 8, 129, 33, True), (3, 4, 300, 70, True),       # one tile of queries and two, two groups of them
    (1, 2, 1500, 40, False), (1, 3, 2500, 200, False),                         # key splits; a second mask of kept rows
])
def test_heads_that_float32_does_not_carry(kind, B, H, L, u, ragged):
    # the second head; the others stay as they are
    w, sel, ub, G = _one_hard_head(kind, B, H, L, u, ragged, 20 + L)
    for fill in ("mean", "value"):
        got, ref, _ = _gradients(w, sel, ub, G, fill)
        _check(got, ref, f"{kind} L{L} u{u} {fill}", [1])
        _check(got, ref, f"beside {kind} L{L} u{u} {fill}", [h for h in range(H) if h != 1])


@pytest.mark.parametrize("B,H,L,u", [(2, 2, 100, 20), (1, 2, 1500, 40), (1, 1, 700, 130)])
def test_infinite_gradients(B, H, L, u):
    # a kept query's dOut is infinite in one element: infinite in that element of dV for every key, as the weights are positive; dQ of
    # that query and dK are not numbers; everything else is as ever
    w = _workload(B, H, L, False, "normal", seed=L)
    sel, ub = _sets(w, u, L)
    G = W.to_f64(W.make_upstream_gradient(w.cfg, 5), "bf16").copy()
    i = int(sel[0, 0, 0])
    G[0, 0, i, 5] = -np.inf
    got, ref, sets = _gradients(w, sel, ub, _bf16(G), "value")
    assert (got[2][0, 0, :, 5] == -np.inf).all() and np.isnan(got[1][0, 0]).all() and np.isnan(got[0][0, 0, i]).all()
    for x in (got, ref):
        for name, t in zip(("dQ", "dK", "dV"), x):
            t[~np.isfinite(t)] = 0.0
    got[1][0, 0], ref[1][0, 0] = 0.0, 0.0
    _check(got, ref, f"infinite L{L}")
