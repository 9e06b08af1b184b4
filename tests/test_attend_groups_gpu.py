"""float32 heads in several query groups of 16: items whose u ends at, before and behind the edge of a group (groups that are
empty in some items)."""
import numpy as np
import pytest

from paper_2106_09236_amd import workloads as W
from tests.test_parity_gpu import check_against_oracle
from tests.test_plan import plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,L", [(24, 4, 750), (7, 3, 750), (46, 4, 640)])
def test_groups_beyond_u(B, H, L):
    p = plan(B, H, L, 12, "f32")
    assert p["attend"] == "key_split" and p["queries_per_group"] == "16" and int(p["query_groups"]) == 3
    cfg = W.small_config("groups", B, H, L, 12, 5.0, "f32", "peaky", True, 1, L)
    w = W.make_workload(cfg, seed=90 + B)
    w.lengths[:7] = [24, 25, 601, 602, L, 0, 1]                       # u = 16, 17, 32, 33, 33 or 34, none, 1
    for b in range(B):
        w.sample_idx[b] = np.minimum(w.sample_idx[b], max(0, int(w.lengths[b]) - 1))
        for x in (w.Q, w.K, w.V):
            x[b, :, int(w.lengths[b]):] = 0
    check_against_oracle(w, label=f"groups B{B} H{H} L{L}")


@pytest.mark.parametrize("fill", ["mean", "value"])
@pytest.mark.parametrize("B,H,L,groups,shares", [
    (1, 4, 1, 32, 4), (1, 1, 33, 32, 4), (16, 5, 32, 32, 2),       # groups of 32, four and two work-groups to a group of queries
    (1, 1, 65, 16, 4), (2, 4, 128, 16, 4), (3, 4, 257, 16, 4),     # groups of 16, four: two tiles and a key, half of the waves, a second step
    (8, 4, 200, 16, 4), (8, 8, 129, 16, 2),                        # ... at most 256 work-groups, and two to a group
])
def test_shared_elements(B, H, L, groups, shares, fill):
    # heads in one key split whose output elements several work-groups share; items of 0, 1 and 2 frames among them
    p = plan(B, H, L, 9, "f32")
    assert p["attend"] == "key_split" and p["merge"] == "none" and int(p["queries_per_group"]) == groups
    assert int(p["element_shares"]) == shares
    assert 2 * B * H * int(p["query_groups"]) <= 256
    cfg = W.small_config("shared", B, H, L, 9, 5.0, "f32", "peaky", B > 1, max(1, L // 2), L)
    w = W.make_workload(cfg, seed=40 + L)
    if B > 2:
        w.lengths[:3] = [0, 1, min(2, L)]
        for b in range(3):
            w.sample_idx[b] = np.minimum(w.sample_idx[b], max(0, int(w.lengths[b]) - 1))
            for x in (w.Q, w.K, w.V):
                x[b, :, int(w.lengths[b]):] = 0
    check_against_oracle(w, label=f"shared B{B} H{H} L{L} {fill}", fill=fill)


@pytest.mark.parametrize("B,H,L,r,lists,length", [(1, 2, 5000, 0.05, 8, 250), (1, 1, 300, 0.3, 5, 64), (2, 2, 700, 0.1, 0, 0)])
@pytest.mark.parametrize("first", [0, 1, 2])
def test_most_of_the_selection_from_one_list(B, H, L, r, lists, length, first):
    # more than 4 candidate lists, whose entries are counted 64 at a time: nearly all selected queries in the first, a middle or
    # the last part of the head, so that one list takes part with all its entries and others with none
    p = plan(B, H, L, 12, "f32", r_sparse=r)
    if lists:
        assert (int(p["lists"]), int(p["list_len"])) == (lists, length)
    w = W.make_workload(W.small_config("onelist", B, H, L, 12, 5.0, "f32", "normal"), seed=70 + first)
    at = (0, L // 2, L - L // 8)[first]
    w.Q[:, :, at:at + L // 8] *= 6
    check_against_oracle(w, label=f"one list L{L} at {at}", r_sparse=r)
