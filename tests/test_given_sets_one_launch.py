"""Calls with given index sets whose attend work-groups form the V column sums themselves: heads at the edges of 4, 8 and 16
loads per thread, padding that must not be read, empty items, and a workspace that holds anything."""
import ctypes

import numpy as np
import pytest

from paper_2106_09236_amd import workloads as W
from tests.test_plan import plan


@pytest.mark.parametrize("dtype,longest,wide", [("f32", 512, 256), ("bf16", 1024, 1024)])
def test_which_calls(dtype, longest, wide):
    for L, own in [(1, "1"), (longest, "1"), (longest + 1, "0")]:
        assert plan(2, 4, L, 4, dtype, u_stride=min(L, 30))["own_sums"] == own
    # however many work-groups, but not where the call selects by itself
    assert plan(600, 1, 64, 4, dtype, u_stride=20)["own_sums"] == "1"
    assert plan(2, 4, 100, 4, dtype)["own_sums"] == "0"
    # float32: one key split where a ticket would bring a launch of its own
    assert plan(16, 4, 512, 32, dtype, u_stride=32)["key_splits"] == "1"


def _check(dtype, B, H, L, u, fill, seed):
    import torch
    from oracle import probsparse_oracle as O
    from paper_2106_09236_amd import binding as psa
    from tests import parity
    w = W.make_workload(W.small_config("own", B, H, L, 4, 5.0, dtype, "normal", B > 1, 1, L), seed=seed)
    if B > 1:
        w.lengths[0], w.lengths[1] = L, 0
    n = w.lengths_or_full()
    rng = np.random.default_rng(seed)
    sel = np.stack([[rng.permutation(L)[:u] for _ in range(H)] for _ in range(B)]).astype(np.int32)
    sets = [[np.unique(sel[b, h][sel[b, h] < n[b]]) for h in range(H)] for b in range(B)]
    ub = np.minimum(u, n).astype(np.int32)
    for b in range(B):                                     # the valid entries first, so that u_b of them are in use
        for h in range(H):
            s = sel[b, h]
            sel[b, h] = np.concatenate([s[s < n[b]], s[s >= n[b]]])
    t = {}
    for k in "QKV":
        x = torch.from_numpy(w.as_f64(k)).to(torch.float32 if dtype == "f32" else torch.bfloat16)
        for b in range(B):
            x[b, :, int(n[b]):] = float("nan")
        t[k] = x.cuda()
    lengths = torch.from_numpy(np.asarray(n, dtype=np.int32)).cuda() if B > 1 else None
    shape = psa.make_shape(B, H, L, 1, psa.PSA_F32 if dtype == "f32" else psa.PSA_BF16)
    ws = torch.full((psa.load().probsparse_attn_with_indices_workspace_bytes(ctypes.byref(shape), u),), 0xFF, dtype=torch.uint8, device="cuda")
    sel_d, u_d = torch.from_numpy(sel).cuda(), torch.from_numpy(ub).cuda()
    outs = [psa.probsparse_attn_fwd_with_indices(t["Q"], t["K"], t["V"], lengths, sel_d, u_d,
                                                 psa.FILL_VALUE if fill == "value" else psa.FILL_MEAN, workspace=ws).float().cpu().numpy()
            for _ in range(2)]
    assert np.array_equal(outs[0], outs[1])
    want = O.attention_with_indices(w.as_f64("Q"), w.as_f64("K"), w.as_f64("V"), w.lengths, sets, fill=fill)
    valid = np.zeros((B, H, L), dtype=bool)
    for b in range(B):
        valid[b, :, :int(n[b])] = True
        assert (outs[0][b, :, int(n[b]):] == 0).all()
    err = parity.output_error(outs[0].astype(np.float64), want, valid)
    assert err <= parity.OUT_TOL[dtype], (dtype, B, H, L, u, fill, err)


@pytest.mark.gpu
@pytest.mark.parametrize("fill", ["mean", "value"])
@pytest.mark.parametrize("dtype,B,H,L,u", [
    ("f32", 1, 1, 1, 1), ("f32", 3, 4, 127, 20), ("f32", 3, 4, 128, 25), ("f32", 3, 4, 129, 25), ("f32", 2, 8, 256, 30), ("f32", 2, 8, 257, 70),
    ("f32", 16, 4, 512, 32), ("f32", 2, 4, 513, 32), ("f32", 4, 4, 512, 256), ("f32", 128, 1, 256, 256), ("f32", 128, 1, 257, 257),
    ("bf16", 1, 1, 1, 1), ("bf16", 3, 4, 255, 28), ("bf16", 3, 4, 257, 28), ("bf16", 2, 8, 512, 40), ("bf16", 2, 8, 513, 40),
    ("bf16", 4, 4, 1024, 35), ("bf16", 2, 4, 1025, 35), ("bf16", 16, 4, 520, 300), ("bf16", 4, 8, 2048, 39),
])
def test_against_oracle(dtype, B, H, L, u, fill):
    _check(dtype, B, H, L, u, fill, 300 + L)
