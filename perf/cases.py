"""Cases of the prob-sparse attention library that are worth timing: what a speech model built on it has it do.

A case is one call of a public entry point of `paper_2106_09236_amd.binding` on inputs that are already on the GPU, on
the current stream:

    kind "fwd"      probsparse_attn_fwd                the attention of one layer, u = ceil(c ln n), mean fill
    kind "opt"      probsparse_attn_fwd_opt            the paper's own choices: u = ceil(r n), v_i for the other rows
    kind "indices"  probsparse_attn_fwd_with_indices   a layer that reuses the index sets of the layer before it
    kind "mhsa"     probsparse_mhsa_fwd                the whole multi-head module with its projections
    kind "bwd"      probsparse_attn_bwd                the gradients of attention and fill for given index sets

Shapes are those of the five workloads of the benchmark spec and of utterances between them (4 or 8 heads of 64, 40 ms frames:
40 to 750 frames for corpus clips, up to 16384 for long-form audio).  `keep` says whether the caller holds on to the
output and the scratch (a serving loop) or lets each call allocate them (a module's forward in a training step).
`len_lo` > 0 is a ragged batch with lengths in [len_lo, len_hi], padded to L.
"""
import math

import torch

from paper_2106_09236_amd import binding as psa

D = 64


def _case(kind, dtype, B, H, L, values, factor=5.0, rule="log", fill="mean", len_lo=0, len_hi=0, keep=True, **name):
    return dict(name, kind=kind, dtype=dtype, B=B, H=H, L=L, U=max(1, math.ceil((5.0 if rule == "ratio" else factor) * math.log(L))), values=values,
                factor=factor, rule=rule, fill=fill, len_lo=len_lo, len_hi=len_hi, keep=keep)


def listed():
    return [
        # one five-second utterance, nothing batched: the smallest call, latency alone
        _case("fwd", "f32", 1, 4, 128, "normal", name="utterance_f32"),
        # an encoder layer of the paper's own model on a batch of 20-second clips
        _case("fwd", "f32", 16, 4, 512, "peaky", name="batch_f32"),
        # corpus clips of up to 30 s in one padded batch: an odd length that is no multiple of any tile
        _case("fwd", "f32", 24, 4, 750, "peaky", len_lo=120, len_hi=750, keep=False, name="ragged_f32"),
        # the same in bfloat16 serving, up to 20 s
        _case("fwd", "bf16", 32, 4, 512, "peaky", len_lo=40, len_hi=500, name="ragged_bf16"),
        # a batch of 80-second segments in an 8-head layer
        _case("fwd", "bf16", 8, 8, 2048, "mixture", name="batch_bf16"),
        # eleven minutes of audio in one sequence
        _case("fwd", "bf16", 1, 8, 16384, "mixture", name="longform_bf16"),
        # half of the queries kept and v_i for the others, as the paper trains and evaluates it
        _case("opt", "bf16", 8, 8, 2048, "mixture", 0.5, "ratio", "value", keep=False, name="ratio_bf16"),
        # a layer that reuses its predecessor's index sets
        _case("indices", "f32", 16, 4, 512, "peaky", name="indices_f32"),
        # the whole module: a single odd utterance, and a large batch
        _case("mhsa", "f32", 1, 4, 333, "normal", name="module_utterance_f32"),
        _case("mhsa", "bf16", 8, 8, 2048, "normal", name="module_batch_bf16"),
        # gradients in retraining: the paper's ratio rule in float32, the logarithmic rule in bfloat16
        _case("bwd", "f32", 16, 4, 512, "peaky", 0.5, "ratio", "value", keep=False, name="backward_ratio_f32"),
        _case("bwd", "bf16", 8, 8, 2048, "mixture", keep=False, name="backward_bf16"),
    ]


def _cost(case):
    """Seconds the case takes at a nominal card's rates (float32 tensors and gradients are computed in float64)."""
    w = work(case)
    return w["bytes"] / 8e12 + w["flops"] / (78.6e12 if case["dtype"] == "f32" or case["kind"] == "bwd" else 2.5e15)


def draw(rng):
    most = max(_cost(c) for c in listed())

    def log_uniform(lo, hi):
        return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))
    while True:
        kind = rng.choice(["fwd"] * 6 + ["opt", "indices", "mhsa", "mhsa", "bwd", "bwd"])
        dtype = rng.choice(["f32", "bf16"])
        L = log_uniform(40, 16384)
        B, H = log_uniform(1, 64), rng.choice([4, 8])
        ratio = kind == "opt" or (kind in ("indices", "bwd") and rng.random() < 0.5)
        ragged = B > 1 and rng.random() < 0.5
        case = _case(kind, dtype, B, H, L, rng.choice(["normal", "peaky", "mixture"]) if kind != "mhsa" else "normal",
                     rng.choice([0.35, 0.4, 0.45, 0.5]) if ratio else rng.choice([3.0, 5.0, 5.0, 5.0]),
                     "ratio" if ratio else "log", "value" if ratio else "mean", max(1, L // 8) if ragged else 0, L if ragged else 0, rng.random() < 0.5)
        # the listed cases hold up to 131072 queries in bfloat16 and 72000 in float32
        if B * H * L <= (131072 if dtype == "bf16" else 72000) and _cost(case) <= most:
            return case


def _kept(case, n):
    """u of an item with n valid frames."""
    u = math.ceil(case["factor"] * (n if case["rule"] == "ratio" else math.log(n))) if n > 1 else 1
    return max(1, min(u, n))


def _values(case, g, n):
    """Q, K, V [B, H, L, 64] float32.  "normal": N(0, 1).  "peaky": the same, but a tenth of the query rows are 4 times a
    valid key row plus noise, so that a few queries have a sharply peaked score distribution.  "mixture": 32 components
    with common centres; a frame picks one for its rows of Q, K and V."""
    B, H, L = case["B"], case["H"], case["L"]
    dev = g.device

    def normal(*shape):
        return torch.randn(shape, generator=g, device=dev)
    if case["values"] == "mixture":
        centres = 2.0 * normal(32, D)
        mid = centres[torch.randint(0, 32, (B, H, L), generator=g, device=dev)]
        return [mid + 0.5 * normal(B, H, L, D) for _ in range(3)] + [torch.zeros((B, H, L), dtype=torch.bool, device=dev)]
    Q, K, V = (normal(B, H, L, D) for _ in range(3))
    peaky = torch.zeros((B, H, L), dtype=torch.bool, device=dev)
    if case["values"] == "peaky":
        peaky = torch.rand((B, H, L), generator=g, device=dev) < 0.1
        key = (torch.rand((B, H, L), generator=g, device=dev) * n.view(B, 1, 1)).long()
        row = torch.gather(K, 2, key.unsqueeze(-1).expand(B, H, L, D))
        Q = torch.where(peaky.unsqueeze(-1), 4.0 * row + 0.1 * normal(B, H, L, D), Q)
    return Q, K, V, peaky


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    B, H, L, U = case["B"], case["H"], case["L"], case["U"]
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    shape = psa.make_shape(B, H, L, U, psa.PSA_F32 if case["dtype"] == "f32" else psa.PSA_BF16)
    rule = psa.U_RATIO if case["rule"] == "ratio" else psa.U_LOG
    fill = psa.FILL_VALUE if case["fill"] == "value" else psa.FILL_MEAN
    s = {"kind": case["kind"], "factor": case["factor"], "rule": rule, "fill": fill, "lengths": None, "out": None, "ws": None}
    n = torch.full((B,), L, dtype=torch.int32, device="cuda")
    if case["len_lo"]:
        n = torch.randint(case["len_lo"], case["len_hi"] + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
        s["lengths"] = n
    valid = torch.arange(L, device="cuda").view(1, L) < n.view(B, 1)                        # [B, L]
    if case["kind"] == "mhsa":
        dm = H * D
        X = torch.randn((B, L, dm), generator=g, device="cuda") * valid.unsqueeze(-1)
        s["X"] = X.to(dtype)
        s["matrices"] = [(torch.randn((dm, dm), generator=g, device="cuda") / math.sqrt(dm)).to(dtype) for _ in range(4)]
        s["biases"] = [(0.1 * torch.randn(dm, generator=g, device="cuda")).to(dtype) for _ in range(4)]
        s["weights"] = psa.make_weights(*s["matrices"], *s["biases"])
    else:
        Q, K, V, peaky = _values(case, g, n)
        pad = valid.view(B, 1, L, 1)
        s["Q"], s["K"], s["V"] = ((t * pad).to(dtype) for t in (Q, K, V))
    if case["kind"] in ("fwd", "opt", "mhsa"):
        idx = (torch.rand((B, H, L, U), generator=g, device="cuda") * n.view(B, 1, 1, 1)).to(torch.int32)
        s["idx"] = torch.minimum(idx, n.view(B, 1, 1, 1) - 1) * valid.view(B, 1, L, 1)
    else:
        # distinct valid queries in no particular order, the peaked ones first
        u = [_kept(case, k) for k in n.tolist()]
        rank = torch.rand((B, H, L), generator=g, device="cuda") + peaky.float()
        rank = rank.masked_fill(~valid.view(B, 1, L), -1.0)
        sel = rank.topk(_kept(case, L), dim=-1).indices.to(torch.int32)
        s["u"] = torch.tensor(u, dtype=torch.int32, device="cuda")
        unused = torch.arange(sel.shape[-1], device="cuda").view(1, 1, -1) >= s["u"].view(B, 1, 1)
        s["sel"] = sel.masked_fill(unused, -1).contiguous()
    if case["kind"] == "bwd":
        s["dOut"] = (torch.randn((B, H, L, D), generator=g, device="cuda") * valid.view(B, 1, L, 1)).to(dtype)
    if case["keep"] and case["kind"] in ("fwd", "opt"):
        s["out"] = torch.empty_like(s["Q"])
        if case["kind"] == "fwd":
            s["ws"] = psa.alloc_workspace(shape, case["factor"])
    elif case["keep"] and case["kind"] == "indices":
        s["out"] = torch.empty_like(s["Q"])
    elif case["keep"] and case["kind"] == "mhsa":
        s["out"] = torch.empty_like(s["X"])
    return s


def run(s):
    kind = s["kind"]
    if kind == "fwd":
        return psa.probsparse_attn_fwd(s["Q"], s["K"], s["V"], s["lengths"], s["idx"], s["factor"], out=s["out"], workspace=s["ws"])
    if kind == "opt":
        return psa.probsparse_attn_fwd_opt(s["Q"], s["K"], s["V"], s["lengths"], s["idx"], s["rule"], s["factor"], s["fill"], out=s["out"], taps=False)
    if kind == "indices":
        return psa.probsparse_attn_fwd_with_indices(s["Q"], s["K"], s["V"], s["lengths"], s["sel"], s["u"], s["fill"], out=s["out"])
    if kind == "mhsa":
        return psa.probsparse_mhsa_fwd(s["X"], s["weights"], s["lengths"], s["idx"], s["rule"], s["factor"], s["fill"], Y=s["out"])
    return psa.probsparse_attn_bwd(s["Q"], s["K"], s["V"], s["lengths"], s["sel"], s["u"], s["dOut"], s["fill"])


def work(case):
    """Inputs read once and outputs written once; the products of the steps themselves.  A ragged batch counts at its mean
    length (padding is written, as zeros, and never read)."""
    B, H, L, U = case["B"], case["H"], case["L"], case["U"]
    size = 4 if case["dtype"] == "f32" else 2
    n = (case["len_lo"] + case["len_hi"]) / 2 if case["len_lo"] else L
    u = _kept(case, max(1, int(n)))
    row, dm = D * size, H * D
    attend = 4 * u * n * D
    if case["kind"] in ("fwd", "opt"):
        return {"bytes": B * H * (3 * n * row + L * row + n * U * 4), "flops": B * H * (2 * D * U * n + attend)}
    if case["kind"] == "indices":
        return {"bytes": B * H * (2 * n * row + u * row + L * row + u * 4), "flops": B * H * attend}
    if case["kind"] == "mhsa":
        return {"bytes": B * (2 * L * dm * size + H * n * U * 4) + 4 * (dm + 1) * dm * size,
                "flops": 8 * B * L * dm * dm + B * H * (2 * D * U * n + attend)}
    # scores and their gradient, then one product for each of dQ, dK, dV
    return {"bytes": B * H * (3 * n * row + u * row + 3 * L * row + u * 4), "flops": B * H * 10 * u * n * D}


def tolerance(case):
    """float32 tensors: sums in float64 (attention) or float32 (projections), one rounding.  bfloat16: one rounding of the
    result; the module also rounds Q, K, V and the attention result to bfloat16, where a last bit decides which queries a
    hard selection keeps, so that single rows of its result may differ as a whole."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    return {"rel": 1e-2, "max": 0.9} if case["kind"] == "mhsa" else {"rel": 1e-2}
