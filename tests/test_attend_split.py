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
