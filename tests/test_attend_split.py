"""How the key-split attend kernel is cut: every key and kept query belongs to exactly one work-group (host plan, no
GPU), and on the GPU the cuts against the oracle: both group sizes, one and several rounds, with and without splits, a
ragged last tile, heads in whole eights (dealt to the XCDs) and not."""
import random

import pytest

from paper_2106_09236_amd import workloads as W
from tests.test_parity_gpu import check_against_oracle
from tests.test_plan import plan


def test_cuts_cover_keys_and_queries_once():
    rng = random.Random(11)
    for _ in range(400):
        L = int(2 ** rng.uniform(0, 15))
        B, H, dtype = int(2 ** rng.uniform(0, 7)), rng.choice([1, 4, 8]), rng.choice(["f32", "bf16"])
        p = plan(B, H, L, 8, dtype, c=rng.choice([0.5, 5.0, 20.0]))
        if p["attend"] != "key_split":
            continue
        nq, groups, splits, rounds, u = (int(p[k]) for k in ("queries_per_group", "query_groups", "key_splits", "rounds", "u_max"))
        assert (groups - 1) * nq < u <= groups * nq
        tiles, per = (L + 31) // 32, rounds * (4 if dtype == "f32" and nq == 32 else 8)      # tiles of 32 keys of one work-group
        assert (splits - 1) * per < tiles <= splits * per
        assert p["merge"] == ("none" if splits == 1 else "last_work_group" if splits <= 8 else "kernel")


@pytest.mark.parametrize("B,H,L,nq,splits,rounds", [
    (1, 4, 333, 16, 1, 2), (2, 4, 1024, 16, 4, 1), (4, 4, 2048, 16, 4, 2), (16, 4, 1000, 16, 1, 4),
    (64, 4, 200, 32, 1, 2), (16, 4, 512, 32, 4, 1), (1, 4, 4096, 32, 32, 1),
])
def test_float32_cuts(B, H, L, nq, splits, rounds):
    p = plan(B, H, L, 32, "f32")
    assert (int(p["queries_per_group"]), int(p["key_splits"]), int(p["rounds"])) == (nq, splits, rounds)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,B,H,L,c", [
    ("f32", 1, 4, 333, 5.0), ("f32", 2, 4, 257, 5.0), ("f32", 3, 4, 700, 5.0), ("f32", 2, 4, 1024, 5.0), ("f32", 1, 8, 545, 3.0),
    ("f32", 9, 8, 289, 5.0), ("f32", 33, 8, 161, 5.0), ("f32", 1, 1, 31, 5.0), ("f32", 1, 2, 4100, 9.0),
    ("bf16", 2, 4, 1500, 5.0), ("bf16", 3, 4, 1500, 5.0), ("bf16", 1, 8, 2300, 5.0),
])
def test_cuts_against_oracle(dtype, B, H, L, c):
    cfg = W.small_config("cuts", B, H, L, 12, c, dtype, "mixture", B > 1, max(1, L // 3), L)
    check_against_oracle(W.make_workload(cfg, seed=900 + L), label=f"B{B} H{H} L{L} c{c} {dtype}")


@pytest.mark.gpu
@pytest.mark.parametrize("B,H,L", [(8, 4, 1041), (2, 4, 333), (8, 4, 1088)])       # rows kernel (odd, whole tiles), key split
@pytest.mark.parametrize("growth", [0.0, 0.13, 0.26, 1.5, -0.5])                    # of the scores, powers of 2 per key
def test_running_maximum_that_lags(B, H, L, growth):
    """Scores that rise along the keys: not at all, by 4 and 8 powers of 2 per tile of 32 keys (the maximum follows in
    some tiles only), in every tile, and never.  bfloat16 results are rounded once: 2^-8 of the row's norm."""
    import torch
    from paper_2106_09236_amd import binding as psa
    g = torch.Generator().manual_seed(L)
    Q, K, V = (0.3 * torch.randn((B, H, L, 64), generator=g) for _ in range(3))
    Q[..., 0] = 8.0
    # q . k = 8 k_0 + ...; in powers of 2 that is k_0 log2(e); a period of 256 keys keeps k_0 exact enough in bfloat16
    K[..., 0] = (torch.arange(L) % 256) * growth / 1.4426950408889634
    Q, K, V = (t.to(torch.bfloat16) for t in (Q, K, V))
    sel = torch.stack([torch.randperm(L, generator=g) for _ in range(B * H)]).reshape(B, H, L).to(torch.int32)
    u = torch.full((B,), L, dtype=torch.int32)
    out = psa.probsparse_attn_fwd_with_indices(Q.cuda(), K.cuda(), V.cuda(), None, sel.cuda(), u.cuda(), psa.FILL_MEAN).cpu().double()
    dense = psa.dense_attn_fwd(Q.cuda(), K.cuda(), V.cuda(), None).cpu().double()
    ref = torch.softmax(Q.double() @ K.double().transpose(-1, -2).contiguous() / 8.0, dim=-1) @ V.double()
    for name, got in (("kept", out), ("dense", dense)):
        err = ((got - ref).norm(dim=-1) / ref.norm(dim=-1)).max().item()
        assert err <= 2.0 ** -8, (name, growth, err)


@pytest.mark.parametrize("B,H,L,chunks_per_wg", [
    (16, 4, 1000, 4), (9, 8, 710, 4), (4, 4, 2048, 2), (2, 4, 1024, 1), (1, 4, 16384, 4),
])
def test_float32_measure_cuts(B, H, L, chunks_per_wg):
    p = plan(B, H, L, 28, "f32")
    assert (p["measure_parts"], p["chunks_per_wg"]) == ("0", str(chunks_per_wg))


def test_static_scratch_admits_what_it_did():
    # near the limit of 16 MiB: shapes whose present cut would need more than the size the workspace has
    from paper_2106_09236_amd import binding as psa
    lib = psa.load()
    limit = lib.probsparse_static_workspace_bytes()
    assert limit == 16 << 20
    for B, H, L, U, c, size in [(227, 8, 12, 8, 5.0, 9655296), (137, 1, 7093, 70, 5.0, 16504320), (167, 4, 977, 40, 3.0, 14128128)]:
        assert int(plan(B, H, L, U, "f32", c=c)["workspace"]) == size <= limit


@pytest.mark.gpu
@pytest.mark.parametrize("B,H,L,U", [(16, 4, 1000, 28), (9, 8, 710, 27), (24, 4, 750, 25), (20, 4, 600, 12), (5, 4, 2100, 9),
                                     (3, 3, 577, 64), (33, 8, 560, 7)])
def test_measure_cuts_against_oracle(B, H, L, U):
    # ragged and whole batches of streamed float32 heads: one to nine chunks per work-group, heads in eights and not
    assert plan(B, H, L, U, "f32")["measure_parts"] == "0"
    for ragged in (False, True):
        cfg = W.small_config("cuts", B, H, L, U, 5.0, "f32", "mixture", ragged, max(1, L // 8), L)
        check_against_oracle(W.make_workload(cfg, seed=700 + L), label=f"B{B} H{H} L{L} ragged={ragged}")


def _busiest_cu(B, H, L, cpw):
    """Most chunks of 64 queries on one CU, float32 streamed measure, all items full: the work-groups of an eighth of
    the heads in order over the 32 CUs of an XCD, the next one to the CU with the least, a quarter for each further one."""
    load = [0.0] * 32
    for first in range(0, (L + 63) // 64, cpw):
        for _ in range((B * H + 7) // 8):
            k = load.index(min(load))
            load[k] += min(cpw, L / 64 - first) + (0.25 if load[k] else 0.0)
    return max(load)


@pytest.mark.parametrize("B,H,L", [(24, 4, 750), (20, 4, 600), (12, 8, 520), (16, 4, 1000), (9, 4, 1700), (5, 4, 3000), (22, 4, 1100),
                                   (40, 4, 900), (1, 2, 9000), (7, 4, 2500), (1, 8, 10000)])
def test_float32_measure_cut_loses_nothing_on_full_batches(B, H, L):
    # against two work-groups per CU in equal shares; calls with and without lengths take the same cut
    two = min(16, (B * H * ((L + 63) // 64) + 511) // 512)
    p = plan(B, H, L, 28, "f32")
    assert p["measure_parts"] == "0"
    assert _busiest_cu(B, H, L, int(p["chunks_per_wg"])) <= _busiest_cu(B, H, L, two)


@pytest.mark.gpu
@pytest.mark.parametrize("B,H,L,c", [(24, 4, 750, 5.0), (7, 4, 2500, 5.0), (9, 4, 1700, 5.0), (24, 4, 750, 15.0)])   # (the last: longer than a chunk)
def test_lists_of_five_chunks(B, H, L, c):
    """Ties across the five chunk lists of a work-group, a head whose measures are all equal, work-groups with a part of
    their chunks or none, and an empty item."""
    import numpy as np
    p = plan(B, H, L, 12, "f32", c=c)
    assert (p["measure"], p["select"], p["chunks_per_wg"]) == ("stream", "lists", "5")
    cfg = W.small_config("five", B, H, L, 12, c, "f32", "peaky", True, 1, L)
    w = W.make_workload(cfg, seed=41 + L)
    w.lengths[0], w.lengths[1], w.lengths[2], w.lengths[3] = L, 321, 257, 0
    for b in range(B):
        n = int(w.lengths[b])
        w.sample_idx[b] = np.minimum(w.sample_idx[b], max(0, n - 1))
    w.Q[0, 0] = 0                                                        # all equal
    for first in (64, 128, 192, 256):                                    # the chunks of a work-group repeat each other
        w.Q[:, 1, first:first + 64] = w.Q[:, 1, :64]
        w.sample_idx[:, 1, first:first + 64] = w.sample_idx[:, 1, :64]
    for b in range(B):                                                   # (padding stays zero)
        w.Q[b, :, int(w.lengths[b]):] = 0
    check_against_oracle(w, label=f"five-{B}-{H}-{L}")


@pytest.mark.gpu
@pytest.mark.parametrize("lengths", [False, True])
@pytest.mark.parametrize("B,H,L", [(24, 4, 750), (12, 8, 520), (9, 4, 1700)])
def test_described_lists_are_what_a_call_with_lengths_makes(B, H, L, lengths):
    # where the plan says that the measure kernel hands on lists, the measure and attend stages alone are the whole call
    import torch
    from paper_2106_09236_amd import binding as psa
    assert plan(B, H, L, 20, "f32")["select"] == "lists"
    g = torch.Generator().manual_seed(L)
    Q, K, V = (torch.randn((B, H, L, 64), generator=g).cuda() for _ in range(3))
    n = torch.randint(L // 6, L + 1, (B,), generator=g, dtype=torch.int32)
    idx = (torch.rand((B, H, L, 20), generator=g) * n.view(B, 1, 1, 1)).to(torch.int32).cuda()
    n = n.cuda() if lengths else None
    ws = psa.alloc_workspace(psa.make_shape(B, H, L, 20, psa.PSA_F32), 5.0).zero_()
    out = torch.zeros_like(Q)
    psa.probsparse_attn_fwd_stages(Q, K, V, n, idx, 5.0, out, ws, psa.STAGE_MEASURE | psa.STAGE_ATTEND)
    assert torch.equal(out, psa.probsparse_attn_fwd(Q, K, V, n, idx, 5.0))


@pytest.mark.gpu
@pytest.mark.parametrize("B,H,L,u", [(1, 2, 64, 2), (16, 8, 512, 512)])      # key split; a wave owns its queries
def test_scores_beyond_the_rounded_maximum(B, H, L, u):
    """float32: at 2^35 the running maximum, rounded to float32, lies 1030 (as a power of 2) below the largest score.  Weights
    overflow: the result is NaN or right, never that of the key whose score is 20 lower."""
    import torch
    from paper_2106_09236_amd import binding as psa
    log2e_scale = 0.125 * 1.4426950408889634
    s = (2.0 ** 35 + 5 * 4096 + 1030) / log2e_scale              # raw score of the best key
    Q, K, V = (torch.zeros((B, H, L, 64)) for _ in range(3))
    Q[..., 0], Q[..., 1] = 2.0 ** 17, 1.0
    high = torch.tensor(s / 2 ** 17).float()
    K[:, :, :2, 0] = high
    K[:, :, 0, 1] = s - float(high) * 2 ** 17
    K[:, :, 1, 1] = K[:, :, 0, 1] - 20 / log2e_scale
    V[:, :, 0], V[:, :, 1] = 1.0, -1.0
    t = ((Q[0, 0, :1].double() @ K[0, 0].double().T) * log2e_scale)[0]
    assert 1025 < float(t[0] - t[0].float().double()) < 1035 and 19 < float(t[0] - t[1]) < 21
    sel = torch.arange(u, dtype=torch.int32).expand(B, H, u).contiguous()
    args = Q.cuda(), K.cuda(), V.cuda(), None
    out = psa.probsparse_attn_fwd_with_indices(*args, sel.cuda(), torch.full((B,), u, dtype=torch.int32).cuda())[:, :, :u].cpu()
    dense = psa.dense_attn_fwd(*args).cpu()
    for got in (out, dense):
        assert bool((got.isnan() | ((got - 1).abs() < 1e-5)).all()), got.flatten()[:4]
