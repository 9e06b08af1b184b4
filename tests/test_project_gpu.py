"""The projections at the edges of their kernels.  bfloat16 tensors with many rows (256 x 128 tiles, several to a work-group)
against the same rows in calls that are too small for that kernel, which tests/test_parity_gpu.py compares with the oracle.  Both add the products of a row in
the same order, so the results are the same bits: no tolerance."""
import pytest
import torch

from paper_2106_09236_amd import binding as psa
from paper_2106_09236_amd import workloads as W
from tests.test_plan import plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,L,H,bias,out", [
    (8, 2048, 8, True, False),     # whole tiles, three per work-group
    (13, 777, 8, False, False),    # a ragged last block of rows, work-groups with one tile and with two
    (4, 8190, 8, True, True),      # the output matrix as well: two rounds; every tile but the first starts inside an item
    (16000, 4, 4, True, True),     # items of 4 frames: 64 to a tile; both launches
    (7, 1100, 15, True, False),    # a ragged last column tile: 960 of 1024 columns
    (64, 2000, 4, False, True),    # ten tiles and more to a work-group
])
def test_many_rows_equal_few_rows(B, L, H, bias, out):
    # `out`: the output matrix takes that kernel as well
    p = plan(B, H, L, 4, "bf16")
    assert p["qkv_project"] == "stream" and (p["out_project"] == "stream") == out
    raw = W.make_mhsa_inputs(1, 1, H, "bf16", 5 + L, bias)
    dev = {k: None if v is None else torch.from_numpy(v.view("int16")).view(torch.bfloat16).cuda() for k, v in raw.items()}
    weights = psa.make_weights(*[dev[k] for k in ("Wq", "Wk", "Wv", "Wo", "bq", "bk", "bv", "bo")])
    g = torch.Generator(device="cuda")
    g.manual_seed(L)
    X = torch.randn((B, L, H * 64), generator=g, device="cuda").to(torch.bfloat16)
    A = torch.randn((B, H, L, 64), generator=g, device="cuda").to(torch.bfloat16)
    many = psa.probsparse_qkv_project(X, weights) + (psa.probsparse_out_project(A, weights),)
    n = max(1, 2000 // L)                     # items per call: at most 2000 rows, or one item cut into such pieces
    p = plan(n, H, min(L, 2000), 4, "bf16")
    assert p["qkv_project"] != "stream" and p["out_project"] != "stream"
    for b in range(0, B, n):
        for l in range(0, L, 2000):
            x, a = X[b:b + n, l:l + 2000].contiguous(), A[b:b + n, :, l:l + 2000].contiguous()
            few = psa.probsparse_qkv_project(x, weights) + (psa.probsparse_out_project(a, weights),)
            for name, m, f in zip("QKV", many, few):
                assert torch.equal(m[b:b + n, :, l:l + 2000], f), (name, b, l)
            assert torch.equal(many[3][b:b + n, l:l + 2000], few[3]), ("Y", b, l)


@pytest.mark.parametrize("B,L,H", [(1, 1, 1), (1, 65, 2), (2, 33, 3), (1, 63, 8),
                                   (1, 2688, 4), (1, 2689, 4)])                    # 504 and 516 work-groups for Q, K and V: the last with two groups and the first with one
def test_few_rows_of_float32(B, L, H):
    # two groups of waves add every other chunk of a contraction.  Against float64, element by element: every product is off by at
    # most 3 * 2^-25 (three bfloat16 parts of a factor, six of nine products) and every addition of at most 6 dm + 2 by 2^-24
    # of the sum of the products' sizes (first order; twice that is allowed)
    p = plan(B, H, L, 4, "f32")
    assert (p["qkv_project"] == "tiles_64x64_two_groups") == (L <= 2688) and p["out_project"] == "tiles_64x64_two_groups"
    dm = H * 64
    g = torch.Generator(device="cuda")
    g.manual_seed(L)
    X = torch.randn((B, L, dm), generator=g, device="cuda")
    A = torch.randn((B, H, L, 64), generator=g, device="cuda")
    Ws = [torch.randn((dm, dm), generator=g, device="cuda") / dm ** 0.5 for _ in range(4)]
    bs = [torch.randn(dm, generator=g, device="cuda") for _ in range(4)]
    weights = psa.make_weights(*Ws, *bs)
    got = psa.probsparse_qkv_project(X, weights) + (psa.probsparse_out_project(A, weights),)
    rows = [X, X, X, A.transpose(1, 2).reshape(B, L, dm)]
    for k, name in enumerate("QKVY"):
        have = got[k].double() if k == 3 else got[k].double().transpose(1, 2).reshape(B, L, dm)
        x, w, b = rows[k].double(), Ws[k].double(), bs[k].double()
        size = x.abs() @ w.abs().T + b.abs()
        assert bool(((have - (x @ w.T + b)).abs() <= 2 * (1.5 + 6 * dm + 2) * 2.0 ** -24 * size).all()), name


@pytest.mark.parametrize("B,L,H", [(1, 1, 1), (1, 65, 2), (2, 33, 3), (1, 63, 4), (3, 50, 5), (1, 333, 8), (1, 130, 15)])
def test_few_rows_of_bfloat16(B, L, H):
    # as many chunks as heads, asked for two ahead.  Against float64: products are exact, each of at most dm + 1 additions is off by
    # at most 2^-24 of the sum of the products' sizes (first order; twice that is allowed), and the result is rounded once (2^-8 between neighbours)
    p = plan(B, H, L, 4, "bf16")
    assert p["qkv_project"] == p["out_project"] == "tiles_64x64"
    dm = H * 64
    g = torch.Generator(device="cuda")
    g.manual_seed(L)

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda").to(torch.bfloat16)
    X, A = normal(B, L, dm), normal(B, H, L, 64)
    Ws, bs = [normal(dm, dm) for _ in range(4)], [normal(dm) for _ in range(4)]
    weights = psa.make_weights(*Ws, *bs)
    got = psa.probsparse_qkv_project(X, weights) + (psa.probsparse_out_project(A, weights),)
    rows = [X, X, X, A.transpose(1, 2).reshape(B, L, dm)]
    for k, name in enumerate("QKVY"):
        have = got[k].double() if k == 3 else got[k].double().transpose(1, 2).reshape(B, L, dm)
        x, w, b = rows[k].double(), Ws[k].double(), bs[k].double()
        want, size = x @ w.T + b, x.abs() @ w.abs().T + b.abs()
        assert bool(((have - want).abs() <= 2 * (dm + 1) * 2.0 ** -24 * size + 2.0 ** -8 * want.abs()).all()), name
