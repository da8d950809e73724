"""The work that is timed on this library: calls a user's program makes through the Python binding.

Every case names one entry point, a shape and the operator's parameters.  The sizes are those of the
workloads and sweeps of this repository (a token-choice router, an expert-choice router, magnitude
pruning, the smooth top-k loss, relaxed ranks) and generic ones between them; `draw` spreads each
kind over its whole range.
"""
from __future__ import annotations

import math

import torch

from paper_2302_01425_amd import binding

P2, P43 = 2.0, 4.0 / 3.0


def _case(kind, op, rows, n, k, p, lam, dist, scale, **more):
    return dict(kind=kind, op=op, rows=rows, n=n, k=k, p=p, lam=lam, dist=dist, scale=scale, **more)


def listed():
    return [
        # one small batch of scores, outputs into buffers the program keeps: a latency-bound call
        dict(name="tiny", **_case("tiny", "mask_jvp", 64, 16, 2, P2, 1.0, "normal", 1.0, keep=True)),
        # training step of a token-choice router: mask and its vector-Jacobian product, tied logits
        dict(name="router", **_case("router", "mask_vjp", 16384, 64, 2, P2, 0.5, "ties", 1.0)),
        # the same with the smooth regulariser and more experts
        dict(name="router smooth", **_case("router_smooth", "mask_jvp", 32768, 128, 8, P43, 1.0, "normal", 2.0)),
        # serving the router: only the chosen experts and their weights come back
        dict(name="dispatch", **_case("dispatch", "sparse", 16384, 64, 2, P2, 0.5, "ties", 1.0, width=8)),
        # smooth top-k loss of a classifier and its gradient (an odd number of classes)
        dict(name="loss", **_case("loss", "loss", 4096, 1001, 5, P43, 1.0, "normal", 2.0)),
        # expert-choice router: every expert picks tokens out of a long row
        dict(name="expert choice", **_case("expert_choice", "mask_jvp", 64, 32768, 1024, P2, 0.1, "normal", 1.0)),
        # forward only (inference) on rows between the one-wavefront and the long ones, ragged
        dict(name="medium rows", **_case("medium", "mask_fwd", 1000, 5001, 501, P2, 0.1, "normal", 1.0)),
        # a tenth of every output unit's weights is kept: top-k in magnitude on matrix rows
        dict(name="prune rows", **_case("prune_rows", "mag_vjp", 4096, 4096, 410, P43, 1e-3, "laplace", 0.02)),
        # a tenth of a whole layer is kept: one row as long as the layer, forward and backward
        dict(name="prune layer", **_case("prune_layer", "mag_vjp", 1, 1 << 24, 1677722, P2, 1e-3, "laplace", 0.02)),
        # a few very long rows with a wide pooled block
        dict(name="long rows", **_case("long", "mask_jvp", 16, 1 << 20, 104858, P2, 0.1, "normal", 1.0)),
        # relaxed ranks of short score lists, differentiated (general weights)
        dict(name="ranks", **_case("ranks", "general_jvp", 4096, 1024, 0, P2, 0.1, "normal", 1.0)),
        # relaxed ranks of long score lists
        dict(name="long ranks", **_case("long_ranks", "general_fwd", 64, 65536, 0, P2, 0.1, "normal", 1.0)),
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, uniform in its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _real(rng, lo, hi):
    return float("%.4g" % math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    kind = rng.choice(("tiny", "router", "router_smooth", "dispatch", "loss", "expert_choice", "medium",
                       "prune_rows", "prune_layer", "long", "ranks", "long_ranks"))
    p = rng.choice((P2, P43))

    def rows_for(n, lo, hi, elements):
        return _log(rng, lo, max(lo, min(hi, elements // n)))

    if kind == "tiny":
        n = rng.randint(2, 64)
        return _case(kind, "mask_jvp", _log(rng, 1, 256), n, rng.randint(1, max(1, n // 4)), p,
                     _real(rng, 0.1, 2.0), "normal", 1.0, keep=True)
    if kind in ("router", "dispatch"):
        n = _log(rng, 8, 256)
        k = rng.randint(1, min(8, n // 4))
        rows = rows_for(n, 1024, 65536, 1 << 22)
        lam = _real(rng, 0.1, 1.0)
        if kind == "router":
            return _case(kind, rng.choice(("mask_vjp", "mask_vjp", "mask_fwd", "masked_value_jvp", "signed_mask_jvp")),
                         rows, n, k, P2, lam, "ties", 1.0)
        return _case(kind, "sparse", rows, n, k, P2, lam, "ties", 1.0, width=min(n, 4 * k))
    if kind == "router_smooth":
        n = _log(rng, 16, 512)
        return _case(kind, rng.choice(("mask_jvp", "mask_vjp")), rows_for(n, 1024, 65536, 1 << 22), n,
                     rng.randint(1, min(16, n // 4)), P43, _real(rng, 0.3, 2.0), "normal", 2.0)
    if kind == "loss":
        n = _log(rng, 10, 4000)
        return _case(kind, "loss", rows_for(n, 128, 8192, 1 << 22), n, rng.randint(1, min(10, n // 2)), p,
                     _real(rng, 0.1, 2.0), "normal", 2.0)
    if kind == "expert_choice":
        n = _log(rng, 4096, 131072)
        return _case(kind, rng.choice(("mask_jvp", "mask_vjp")), rows_for(n, 8, 256, 1 << 22), n,
                     n // rng.randint(8, 64), p, _real(rng, 0.01, 0.2), "normal", 1.0)
    if kind == "medium":
        n = _log(rng, 1025, 8192)
        return _case(kind, rng.choice(("mask_fwd", "mask_jvp")), rows_for(n, 64, 4096, 1 << 23), n, -(-n // 10), p,
                     _real(rng, 0.01, 0.2), "normal", 1.0)
    if kind == "prune_rows":
        n = _log(rng, 256, 16384)
        return _case(kind, rng.choice(("mag_vjp", "mag_fwd")), rows_for(n, 256, 8192, 1 << 24), n, -(-n // 10), p,
                     _real(rng, 1e-4, 1e-2), "laplace", 0.02)
    if kind == "prune_layer":
        n = _log(rng, 1 << 17, 1 << 24)
        return _case(kind, rng.choice(("mag_vjp", "mag_fwd")), 1, n, -(-n // rng.choice((2, 5, 10, 20))), p,
                     _real(rng, 1e-4, 3e-3), "laplace", 0.02)
    if kind == "long":
        n = _log(rng, 1 << 17, 1 << 22)
        return _case(kind, rng.choice(("mask_jvp", "mask_fwd")), rows_for(n, 1, 64, 1 << 24), n, -(-n // 10), p,
                     _real(rng, 0.01, 0.1), "normal", 1.0)
    if kind == "ranks":
        n = _log(rng, 16, 1024)
        return _case(kind, rng.choice(("general_jvp", "general_fwd")), rows_for(n, 64, 8192, 1 << 22), n, 0, P2,
                     _real(rng, 1e-3, 1.0), "normal", 1.0)
    n = _log(rng, 1100, 131072)
    return _case(kind, "general_fwd", rows_for(n, 4, 256, 1 << 22), n, 0, P2, _real(rng, 1e-3, 1.0), "normal", 1.0)


def _values(case, gen):
    rows, n, scale = case["rows"], case["n"], case["scale"]
    dev = torch.device("cuda")
    if case["dist"] == "laplace":
        u = torch.rand((rows, n), generator=gen, device=dev, dtype=torch.float32).clamp_(1e-7, 1.0 - 1e-7) - 0.5
        return (u.sign() * torch.log1p(-2.0 * u.abs()) * -scale).contiguous()
    x = torch.randn((rows, n), generator=gen, device=dev, dtype=torch.float32) * scale
    if case["dist"] == "ties":
        # some entries of a row take the value of another entry: exact ties
        m = max(1, n // 20)
        at = torch.rand((rows, n), generator=gen, device=dev).topk(2 * m, dim=1).indices
        x.scatter_(1, at[:, :m], x.gather(1, at[:, m:]))
    return x.contiguous()


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    rows, n, op = case["rows"], case["n"], case["op"]
    s = {"case": case, "x": _values(case, gen)}
    if op.endswith("jvp") or op.endswith("vjp"):
        s["t"] = torch.randn((rows, n), generator=gen, device="cuda", dtype=torch.float32)
    if op == "loss":
        # the wanted classes, one in every row, as a 0/1 array
        label = torch.randint(0, n, (rows, 1), generator=gen, device="cuda")
        s["t"] = torch.zeros((rows, n), device="cuda", dtype=torch.float32).scatter_(1, label, 1.0)
    if op.startswith("general"):
        s["x"] = -s["x"]                                            # ranks of theta: input -theta
        s["w"] = torch.arange(n, 0, -1, dtype=torch.float32, device="cuda")
    if case.get("keep"):
        s["out"], s["d"] = torch.empty_like(s["x"]), torch.empty_like(s["x"])
    return s


def run(s):
    c = s["case"]
    x, k, p, lam, op = s["x"], c["k"], c["p"], c["lam"], c["op"]
    if op == "mask_jvp":
        return binding.topk_mask_jvp(x, s["t"], k, p, lam, out=s.get("out"), jvp_out=s.get("d"))
    if op == "mask_vjp":
        return binding.topk_mask_vjp(x, s["t"], k, p, lam)
    if op == "mask_fwd":
        return binding.topk_mask_fwd(x, k, p, lam)
    if op == "mag_vjp":
        return binding.topkmag_vjp(x, s["t"], k, p, lam)
    if op == "mag_fwd":
        return binding.topkmag_fwd(x, k, p, lam)
    if op == "masked_value_jvp":
        return binding.topk_masked_value_jvp(x, s["t"], k, p, lam)
    if op == "signed_mask_jvp":
        return binding.topk_signed_mask_jvp(x, s["t"], k, p, lam)
    if op == "loss":
        return binding.topk_mask_loss(x, s["t"], k, p, lam)
    if op == "sparse":
        return binding.topk_mask_sparse_fwd(x, k, p, lam, c["width"])
    if op == "general_jvp":
        return binding.topk_general_jvp(x, s["w"], s["t"], binding.TOPK_PHI_IDENTITY, p, lam)
    return binding.topk_general_fwd(x, s["w"], binding.TOPK_PHI_IDENTITY, p, lam)


def work(case):
    """Bytes: every input read once, every output written once.  Operations: a handful per element
    (compare, classify, output); the path has no contraction."""
    rows, n, op = case["rows"], case["n"], case["op"]
    e = 4.0 * rows * n
    if op == "loss":
        b = 3 * e + 4.0 * rows
    elif op == "sparse":
        b = e + 8.0 * rows * case["width"] + 4.0 * rows
    elif op.startswith("general"):
        b = (4 if op.endswith("jvp") else 2) * e + 4.0 * n
    else:
        b = (4 if op.endswith("vp") else 2) * e
    return {"bytes": b, "flops": 10.0 * rows * n}


def tolerance(case):
    # float32 outputs of float64 decisions: the error of an output is its rounding and that of a few
    # float32 operations on differences of inputs.  Against the same operators in float64 the listed
    # and 30 drawn cases are off by 1e-9 to 1.0e-7 (largest: the mask with p = 4/3 on few pooled
    # entries); the permutation of the compact output does not depend on rounding.
    return {"rel": 4e-7, "differ": 0.0} if case["op"] == "sparse" else {"rel": 4e-7}
