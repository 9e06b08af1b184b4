"""The backward of float32 tensors in full batches, whose work-groups may take 128 keys on 8 waves, and with heads in eights, whose work-groups are dealt to the XCDs head by head, and with one head
less or more: every head's rows must come from its own work-groups."""
import numpy as np
import pytest
import torch

import tests.test_backward_tiles_gpu as tiles
from paper_2106_09236_amd import binding as psa
from paper_2106_09236_amd import workloads as W
from tests.test_backward_gpu import check_backward
from tests.test_plan import plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,L,u", [
    (1, 7, 130, 40), (1, 8, 130, 40), (3, 3, 130, 40), (2, 8, 40, 20),   # one or two groups of queries, blocks of 32 keys
    (6, 4, 700, 70), (5, 5, 700, 70),                                    # key splits and their partial sums
    (1, 8, 1700, 850), (1, 9, 1700, 850),                                # dQ from a kernel of its own
])
def test_heads_in_eights(B, H, L, u):
    tiles.test_tiles("f32", B, H, L, u)


@pytest.mark.parametrize("fill", ["mean", "value"])
@pytest.mark.parametrize("B,H,L,u,keys", [
    (8, 8, 512, 256, 128), (16, 4, 511, 70, 128), (16, 4, 385, 300, 128), (8, 8, 1024, 768, 128),     # four and eight blocks of 128 keys a head
    (32, 8, 128, 100, 128), (32, 8, 127, 70, 128), (64, 4, 65, 65, 128),  # one block: dQ goes straight to memory
    (64, 4, 200, 100, 128), (16, 8, 129, 129, 128), (16, 16, 1000, 20, 128),      # two blocks, one key in the second, several blocks to a work-group
    (16, 4, 511, 17, 64), (32, 8, 128, 64, 64), (32, 8, 127, 15, 64), (64, 4, 65, 33, 64), (32, 8, 129, 32, 64),   # few kept queries: blocks of 64
])
def test_full_batches(B, H, L, u, keys, fill):
    # calls without lengths: blocks of 128 keys on 8 waves, where they fill the chip
    assert int(plan(B, H, L, 4, "f32", u_stride=u)["backward_keys_no_lengths"]) == keys
    w = W.make_workload(W.small_config("full", B, H, L, 4, 5.0, "f32", "mixture"), seed=500 + L + u)
    r = np.random.Generator(np.random.PCG64(L + u))
    ub = min(u, L)
    sel = np.full((B, H, u), -1, dtype=np.int32)
    for b in range(B):
        for h in range(H):
            sel[b, h, :ub] = r.permutation(L)[:ub]
            sel[b, h, 6:ub:7] = -1
    check_backward(w, torch.from_numpy(sel).cuda(), torch.full((B,), ub, dtype=torch.int32, device="cuda"), fill, label=f"full B{B} H{H} L{L} u{u} {fill}")


@pytest.mark.parametrize("B,H,L,u", [
    (32, 8, 128, 100), (64, 4, 65, 65),                                  # one block of 128 keys: dQ goes straight to memory
    (16, 4, 512, 256), (16, 8, 129, 129), (4, 8, 996, 100),              # one block a split
    (8, 8, 1024, 512), (8, 8, 871, 40), (8, 8, 1946, 60), (8, 8, 1702, 100),      # two and four, also with an odd number of the smaller splits
    (4, 8, 2907, 17), (8, 8, 2225, 40), (16, 8, 1702, 33),               # three, five and seven: a split's halves meet within a block
    (32, 8, 1302, 20),                                                   # eleven, all in one split
])
def test_full_lengths_give_the_same_bits(B, H, L, u):
    # lengths that are all L and no lengths: blocks of 64 keys and of 128, whose sums are formed in the same order
    p = plan(B, H, L, 4, "f32", u_stride=u)
    assert (p["backward_keys"], p["backward_keys_no_lengths"]) == ("64", "128")
    g = torch.Generator(device="cuda")
    g.manual_seed(L + u)
    Q, K, V, G = (torch.randn((B, H, L, 64), generator=g, device="cuda") for _ in range(4))
    # half of a key's elements with much in common, which cancels in dQ: sums in another order differ in float32 bits there
    Q[..., :32] = 0.0
    K[..., :32] += 30000.0
    sel = torch.rand((B, H, L), generator=g, device="cuda").topk(u, dim=-1).indices.to(torch.int32).contiguous()
    ub = torch.full((B,), u, dtype=torch.int32, device="cuda")
    full = torch.full((B,), L, dtype=torch.int32, device="cuda")
    for fill in (psa.FILL_MEAN, psa.FILL_VALUE):
        none = psa.probsparse_attn_bwd(Q, K, V, None, sel, ub, G, fill)
        same = psa.probsparse_attn_bwd(Q, K, V, full, sel, ub, G, fill)
        for name, a, b in zip(("dQ", "dK", "dV"), none, same):
            assert torch.equal(a, b), (name, int((a != b).sum()))
