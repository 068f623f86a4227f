"""The work this library is measured by: the products and the packing that a
user's program has it do, from one decode token to a 4096-row prefill.

A case names one call:
  op     "run"       nmspmm_run
         "ex"        nmspmm_run_ex with alpha = M/N, a bias and an activation
         "ws"        nmspmm_run_ws with a workspace of nmspmm_workspace_bytes
         "compress"  nmspmm_compress_device
  m, k, n, N, M, V   the shape and the pattern
  dist   "uniform": A and B from U[-1, 1]; "normal": A ~ N(0, 1), B ~ N(0, 0.02^2)
  act    the activation of "ex"
Shapes and distributions are those of nm_workloads.py (the named runs R1 to R5
and the shape x sparsity sweep) and sizes around them.
"""
import math

import torch

import paper_2503_01253_amd as nm

LEVELS = ((16, 32), (12, 32), (8, 32), (4, 32), (32, 32), (4, 16), (2, 4))
LARGEST = 2.0 * 4096 * 4096 * 2048    # useful flops of the largest listed case


def _case(name, op, m, k, n, N, M, V, dist, act="none"):
    return dict(name=name, op=op, m=m, k=k, n=n, N=N, M=M, V=V, dist=dist, act=act)


def listed():
    return [
        # the smallest square product of the workloads (R1): launch latency counts
        _case("square_256_50", "run", 256, 256, 256, 16, 32, 32, "uniform"),
        # decoding one sequence: one token through a sparse 8192 x 8192 layer
        _case("decode_1", "run", 1, 8192, 8192, 4, 32, 64, "normal"),
        # decoding 16 sequences at once (R5a)
        _case("decode_16", "run", 16, 8192, 8192, 4, 32, 64, "normal"),
        # a serving loop that keeps its own workspace, 64 sequences (R5b)
        _case("decode_64_ws", "ws", 64, 8192, 8192, 4, 32, 64, "normal"),
        # 128 rows, the workspace left to the library (R5c)
        _case("decode_128", "run", 128, 8192, 8192, 4, 32, 64, "normal"),
        # an odd batch through an MLP up-projection, bias and GELU fused
        _case("mlp_37_gelu", "ex", 37, 4096, 11008, 8, 32, 32, "normal", "gelu"),
        # a medium square product at 62.5 % sparsity (C-12 of the sweep)
        _case("medium_512_62", "run", 512, 2048, 2048, 12, 32, 32, "uniform"),
        # a prompt of odd length through a layer whose width fits no tile
        _case("prefill_1111", "run", 1111, 4096, 4192, 16, 32, 32, "normal"),
        # prefill of 2048 tokens through an MLP up-projection (R4), bias and ReLU fused
        _case("mlp_2048_relu", "ex", 2048, 4096, 11008, 8, 32, 32, "normal", "relu"),
        # the headline product at 50 % sparsity (R2), and the sparsest level (R3d)
        _case("square_4096_50", "run", 4096, 4096, 4096, 16, 32, 32, "uniform"),
        _case("square_4096_87", "run", 4096, 4096, 4096, 4, 32, 64, "uniform"),
        # pruning a layer's weight on the GPU
        _case("compress_mlp_75", "compress", 1, 4096, 11008, 8, 32, 32, "normal"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(("run", "run", "run", "ex", "ws", "ws", "compress"))
    while True:
        N, M = rng.choice(LEVELS)
        V = rng.choice((16, 32, 32, 32, 64, 64, 128))
        m = 1 if op == "compress" else _log(rng, 1, 4096)
        k = max(1, _log(rng, 256, 11008) // 32) * 32
        n = max(1, _log(rng, 256, 11008) // V) * V
        if 2.0 * m * n * (k // M) * N <= LARGEST:
            break
    act = rng.choice(("none", "relu", "gelu")) if op == "ex" else "none"
    return dict(op=op, m=m, k=k, n=n, N=N, M=M, V=V, dist=rng.choice(("uniform", "normal")), act=act)


def _values(gen, rows, cols, dist, scale):
    if dist == "uniform":
        return torch.rand(rows, cols, generator=gen, device="cuda") * 2 - 1
    return torch.randn(rows, cols, generator=gen, device="cuda") * scale


def _inputs(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    m, k, n, N, M, V = (case[x] for x in ("m", "k", "n", "N", "M", "V"))
    if case["op"] == "compress":
        return {"B": _values(gen, k, n, case["dist"], 0.02)}
    w, q = (k // M) * N, n // V
    keep = torch.rand(k // M, q, M, generator=gen, device="cuda").argsort(-1)[..., :N].sort(-1).values
    s = {"A": _values(gen, m, k, case["dist"], 1.0), "Bc": _values(gen, w, n, case["dist"], 0.02),
         "idx": keep.permute(0, 2, 1).reshape(w, q).to(torch.uint8).contiguous(), "bias": None}
    if case["op"] == "ex":
        s["bias"] = torch.randn(n, generator=gen, device="cuda")
    return s


def prepare(case, seed):
    m, k, n, N, M, V = (case[x] for x in ("m", "k", "n", "N", "M", "V"))
    s = _inputs(case, seed)
    s.update(case=dict(case), shape=(m, n, k, N, M, V))
    if case["op"] == "compress":
        w = (k // M) * N
        s["Bc"] = torch.empty(w, n, device="cuda")
        s["idx"] = torch.empty(w, n // V, dtype=torch.uint8, device="cuda")
        return s
    s["C"] = torch.empty(m, n, device="cuda")
    if case["op"] == "ws":
        size = nm.nmspmm_workspace_bytes(m, n, k, N, M, V)
        s["workspace"] = torch.empty(size, dtype=torch.uint8, device="cuda") if size > 0 else None
    return s


def run(s):
    case = s["case"]
    if case["op"] == "compress":
        return nm.nmspmm_compress_device(s["B"], s["Bc"], s["idx"], case["N"], case["M"], case["V"])
    if case["op"] == "ex":
        return nm.nmspmm_run_ex(s["A"], s["Bc"], s["idx"], s["C"], *s["shape"], alpha=case["M"] / case["N"],
                                bias=s["bias"], act=case["act"])
    if case["op"] == "ws":
        return nm.nmspmm_run_ws(s["A"], s["Bc"], s["idx"], s["C"], *s["shape"], s["workspace"])
    return nm.nmspmm_run(s["A"], s["Bc"], s["idx"], s["C"], *s["shape"])


def work(case):
    m, k, n, N, M, V = (case[x] for x in ("m", "k", "n", "N", "M", "V"))
    w, q = (k // M) * N, n // V
    if case["op"] == "compress":
        return {"bytes": 4 * k * n + 4 * w * n + w * q, "flops": 2 * k * n}
    bias = 4 * n if case["op"] == "ex" else 0
    return {"bytes": 4 * m * k + 4 * w * n + w * q + 4 * m * n + bias, "flops": 2 * m * n * w}


def tolerance(case):
    if case["op"] == "compress":
        return "exact"
    # fp32 sums of w terms: two summation orders differ by about 2e-8 * sqrt(w)
    # (8.3e-7, largest 8.3e-6, at w = 2048; 1.1e-7 at w = 128), four times that
    w = case["k"] // case["M"] * case["N"]
    rel = max(8e-7, 8e-8 * math.sqrt(w))
    return {"rel": rel, "max": 10 * rel}


def exact(case, seed):
    m, k, n, N, M, V = (case[x] for x in ("m", "k", "n", "N", "M", "V"))
    s = _inputs(case, seed)
    if case["op"] == "compress":
        # the N rows of largest squared norm per window and column block, in order
        B = s["B"].view(k // M, M, n // V, V)
        norms = B.double().square().sum(-1).permute(0, 2, 1)                    # window, block, row
        keep = norms.sort(dim=-1, descending=True, stable=True).indices[..., :N].sort(-1).values
        keep = keep.permute(0, 2, 1)                                            # window, kept row, block
        rows = torch.take_along_dim(B, keep[..., None], dim=1)
        return (rows.reshape(-1, n).double(), keep.reshape(-1, n // V).to(torch.uint8))
    w = (k // M) * N
    window = torch.arange(w, device="cuda")[:, None] // N * M
    at = (window + s["idx"].long()).repeat_interleave(V, dim=1)
    B = torch.zeros(k, n, dtype=torch.float64, device="cuda").scatter_(0, at, s["Bc"].double())
    C = s["A"].double() @ B
    if case["op"] == "ex":
        C = C * (M / N) + s["bias"].double()
        if case["act"] == "relu":
            C = C.clamp_min(0)
        elif case["act"] == "gelu":
            C = 0.5 * C * (1 + torch.erf(C / math.sqrt(2)))
    return C
