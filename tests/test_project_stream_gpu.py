"""The projections of bfloat16 tensors with many rows (256 x 128 tiles, several to a work-group) against the same rows in calls
that are too small for that kernel, which tests/test_parity_gpu.py compares with the oracle.  Both add the products of a row in
the same order, so the results are the same bits: no tolerance."""
import pytest
import torch

from paper_2106_09236_amd import binding as psa
from paper_2106_09236_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,L,H,bias", [
    (8, 2048, 8, True),            # whole tiles, three per work-group
    (13, 777, 8, False),           # a ragged last block of rows, work-groups with one tile and with two
    (4, 8190, 8, True),            # the output matrix as well: two rounds; every tile but the first starts inside an item
    (16000, 4, 4, True),           # items of 4 frames: 64 to a tile; both launches
    (7, 1100, 15, True),           # a ragged last column tile: 960 of 1024 columns
    (64, 2000, 4, False),          # ten tiles and more to a work-group
])
def test_many_rows_equal_few_rows(B, L, H, bias):
    raw = W.make_mhsa_inputs(1, 1, H, "bf16", 5 + L, bias)
    dev = {k: None if v is None else torch.from_numpy(v.view("int16")).view(torch.bfloat16).cuda() for k, v in raw.items()}
    weights = psa.make_weights(*[dev[k] for k in ("Wq", "Wk", "Wv", "Wo", "bq", "bk", "bv", "bo")])
    g = torch.Generator(device="cuda")
    g.manual_seed(L)
    X = torch.randn((B, L, H * 64), generator=g, device="cuda").to(torch.bfloat16)
    A = torch.randn((B, H, L, 64), generator=g, device="cuda").to(torch.bfloat16)
    many = psa.probsparse_qkv_project(X, weights) + (psa.probsparse_out_project(A, weights),)
    n = max(1, 2000 // L)                     # items per call: at most 2000 rows, or one item cut into such pieces
    for b in range(0, B, n):
        for l in range(0, L, 2000):
            x, a = X[b:b + n, l:l + 2000].contiguous(), A[b:b + n, :, l:l + 2000].contiguous()
            few = psa.probsparse_qkv_project(x, weights) + (psa.probsparse_out_project(a, weights),)
            for name, m, f in zip("QKV", many, few):
                assert torch.equal(m[b:b + n, :, l:l + 2000], f), (name, b, l)
            assert torch.equal(many[3][b:b + n, l:l + 2000], few[3]), ("Y", b, l)
