"""The work whose speed this repository is judged by: calls of the C ABI as a
training step or a serving loop makes them, through the Python binding.

Five kinds of call:

  gemm     compass_gemm: C = A W^T (+ an fp32 partial), one bf16 rounding
  noalloc  compass_gemm_noalloc: the same for callers that cannot allocate
  ag       compass_ag_gemm: fused AllGather + GEMM of one tensor-parallel rank
  rs       compass_gemm_rs: fused GEMM + ReduceScatter with sends
  decomp   compass_decomp_gemm: either pattern as d pipelined sub-operators

Shapes are one tensor-parallel rank's share of a transformer layer (the
evaluation configurations of `synth`, and the ragged shapes of the tests).
Link rates are in GB/s per ring direction, 0 for links as fast as the copy
engines go. All operands are bf16 with fp32 partial sums.
"""
from __future__ import annotations

import math

import torch

from paper_2609_10549_amd import compass as C


def _gemm(name, kind, M, N, K, partial):
    return {"name": name, "kind": kind, "M": M, "N": N, "K": K, "partial": partial}


def _fused(name, kind, M, N, K, n, rank, ring, fwd, bwd, d=1, pattern=""):
    return {"name": name, "kind": kind, "M": M, "N": N, "K": K, "n": n, "rank": rank, "ring": ring,
            "fwd": fwd, "bwd": bwd, "d": d, "pattern": pattern}


def listed():
    return [
        # the smallest fused call (two ranks, 512 tokens): launch and copy latency
        _fused("ag_tp2_small", "ag", 512, 1024, 512, 2, 0, "single", 0, 0),
        # a serving step of a QKV projection: a few dozen tokens against one rank's weight
        _gemm("noalloc_serve_qkv", "noalloc", 48, 3072, 8192, False),
        # odd sizes: no dimension a multiple of a tile, an fp32 partial added
        _gemm("gemm_ragged_partial", "gemm", 1000, 776, 4104, True),
        # a short prompt through an MLP's first projection
        _gemm("gemm_prompt_fc1", "gemm", 640, 2048, 4096, False),
        # the QKV projection of 4096 tokens: neither 256 x 256 nor 128 x 128 tiles fill whole waves
        _gemm("gemm_qkv", "gemm", 4096, 3072, 8192, False),
        # an MLP's second projection with the incoming fp32 partial sum
        _gemm("gemm_fc2_partial", "gemm", 8192, 4096, 2048, True),
        # the largest projection, alone (a step without tensor parallelism's copies)
        _gemm("gemm_gpt3", "gemm", 8192, 6144, 12288, False),
        # the MLP pair of an 8-way layer, links as fast as the copy engines go
        _fused("ag_fc1", "ag", 8192, 2048, 4096, 8, 0, "double", 0, 0),
        _fused("rs_fc2", "rs", 8192, 4096, 2048, 8, 0, "single", 0, 0),
        # the QKV projection as four pipelined sub-operators
        _fused("decomp_qkv_d4", "decomp", 4096, 3072, 8192, 8, 0, "single", 280, 0, 4, "ag"),
        # the largest pair, the two ring directions at 4 : 1
        _fused("ag_gpt3", "ag", 8192, 6144, 12288, 8, 0, "double", 396, 99),
        _fused("rs_gpt3", "rs", 8192, 12288, 6144, 8, 0, "double", 710, 177.5),
    ]


_FLOPS_MAX = 1.2e12          # the largest listed call
_LINK_BYTES_MAX = 330e6      # what its links carry into one rank


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _step(v, s):
    return max(s, int(round(v / s)) * s)


def _dim(rng, lo, hi):
    """A column count or depth: half of them whole tiles, half any multiple of 8."""
    return _step(_log(rng, lo, hi), rng.choice((8, 128)))


def draw(rng):
    while True:
        kind = rng.choice(("gemm", "gemm", "noalloc", "ag", "rs", "decomp"))
        N, K = _dim(rng, 256, 12288), _dim(rng, 256, 12288)
        if kind in ("gemm", "noalloc"):
            M = int(_log(rng, 1, 8192))
            if 2.0 * M * N * K > _FLOPS_MAX:
                continue
            return {"kind": kind, "M": M, "N": N, "K": K, "partial": rng.random() < 0.35}
        pattern = kind if kind != "decomp" else rng.choice(("ag", "rs"))
        n = rng.choice((2, 4, 8))
        ring = rng.choice(("single", "double"))
        d = rng.choice((2, 4)) if kind == "decomp" else 1
        M = _step(_log(rng, 256, 8192), 2 * n * d * rng.choice((1, 8)))
        if M > 8192 or 2.0 * M * N * K > _FLOPS_MAX:
            continue
        moved = M * (n - 1) / n * (K * 2 if pattern == "ag" else N * 4)
        if moved > _LINK_BYTES_MAX:
            continue
        fwd = bwd = 0
        if rng.random() < 0.5:   # paced: the transfer about as long as the GEMM
            want = moved / (2.0 * M * N * K / 1e15 + 20e-6) / 1e9 / rng.uniform(0.8, 1.6)
            if ring == "single":
                fwd = round(min(max(want, 40.0), 400.0), 1)
            else:
                bwd = round(min(max(want / 2, 20.0), 180.0), 1)
                fwd = round(bwd * rng.choice((1, 2, 4)), 1)
        return {"kind": kind, "M": M, "N": N, "K": K, "n": n, "rank": rng.randrange(n), "ring": ring,
                "fwd": fwd, "bwd": bwd, "d": d, "pattern": pattern if kind == "decomp" else ""}


def _pattern(case):
    return case["pattern"] if case["kind"] == "decomp" else case["kind"]


def _inputs(case, seed):
    """Activations N(0, 1), weights N(0, 0.02), partial sums N(0, 1)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    M, N, K = case["M"], case["N"], case["K"]
    A = torch.randn((M, K), generator=g, device="cuda", dtype=torch.bfloat16)
    W = torch.randn((N, K), generator=g, device="cuda", dtype=torch.bfloat16).mul_(0.02)
    P = None
    if case.get("partial") or _pattern(case) == "rs":
        P = torch.randn((M, N), generator=g, device="cuda", dtype=torch.float32)
    return A, W, P


def prepare(case, seed):
    A, W, P = _inputs(case, seed)
    M, N, K, kind = case["M"], case["N"], case["K"], case["kind"]
    out = torch.zeros((M, N), dtype=torch.bfloat16, device="cuda")
    if kind in ("gemm", "noalloc"):
        return {"kind": kind, "A": A, "W": W, "P": P, "C": out}
    n, rank, rows = case["n"], case["rank"], M // case["n"]
    s = {"kind": kind, "pattern": _pattern(case), "d": case["d"], "C": out,
         "links": C.links(case["fwd"] * 1e9, case["bwd"] * 1e9)}
    if s["pattern"] == "ag":
        # the rank's own shard is in place; the others' live in buffers of their own
        gathered = torch.zeros((M, K), dtype=torch.bfloat16, device="cuda")
        gathered[rank * rows:(rank + 1) * rows] = A[rank * rows:(rank + 1) * rows]
        shards = [gathered[q * rows:(q + 1) * rows] if q == rank else A[q * rows:(q + 1) * rows].clone()
                  for q in range(n)]
        s["problem"] = C.ag_problem(shards, gathered, W, out, rank, case["ring"])
        s["keep"] = (W, shards)
        s["gathered"] = gathered
    else:
        parts = [P[q * rows:(q + 1) * rows].clone() for q in range(n)]
        stage = torch.zeros((M, N), dtype=torch.float32, device="cuda")
        sends = [None if q == rank else torch.zeros((rows, N), dtype=torch.bfloat16, device="cuda")
                 for q in range(n)]
        s["problem"] = C.rs_problem(A, W, parts, stage, out, sends, rank, case["ring"])
        s["keep"] = (A, W, parts, stage)
        s["sends"] = sends
    return s


def run(state):
    kind = state["kind"]
    if kind == "gemm":
        C.compass_gemm(state["A"], state["W"], state["C"], state["P"])
        return state["C"]
    if kind == "noalloc":
        C.compass_gemm_noalloc(state["A"], state["W"], state["C"], state["P"])
        return state["C"]
    if kind == "decomp":
        C.compass_decomp_gemm(state["problem"], state["d"], state["links"])
    elif kind == "ag":
        C.compass_ag_gemm(state["problem"], state["links"])
    else:
        C.compass_gemm_rs(state["problem"], state["links"])
    if state["pattern"] == "ag":
        return {"C": state["C"], "gathered": state["gathered"]}
    return {"C": state["C"], "sends": [x for x in state["sends"] if x is not None]}


def work(case):
    """Operands read once, results written once. An AllGather also writes the
    gathered rows of the other ranks; a ReduceScatter reads every fp32 partial
    and writes the other ranks' chunks a second time, to their destinations."""
    M, N, K = case["M"], case["N"], case["K"]
    b = 2 * (M * K + N * K + M * N)
    if case["kind"] in ("gemm", "noalloc"):
        b += 4 * M * N if case["partial"] else 0
    elif _pattern(case) == "ag":
        b += 2 * M * K * (case["n"] - 1) // case["n"]
    else:
        b += 4 * M * N + 2 * M * N * (case["n"] - 1) // case["n"]
    return {"bytes": b, "flops": 2.0 * M * N * K}


def tolerance(case):
    """fp32 accumulation and one rounding to bf16: against 64 bits the result
    is 1.66e-3 off (2-norm) and at most half a unit in the last place (2^-8 of
    the value); four times that."""
    return {"rel": 6.6e-3, "max": 1.6e-2}


def exact(case, seed):
    A, W, P = _inputs(case, seed)
    Wt = W.double().t().contiguous()
    out = torch.empty((case["M"], case["N"]), dtype=torch.float64, device="cuda")
    for r in range(0, case["M"], 1024):
        torch.matmul(A[r:r + 1024].double(), Wt, out=out[r:r + 1024])
    if P is not None:
        out += P.double()
    if case["kind"] in ("gemm", "noalloc"):
        return out
    if _pattern(case) == "ag":
        return {"C": out, "gathered": A.double()}
    rows = case["M"] // case["n"]
    return {"C": out, "sends": [out[q * rows:(q + 1) * rows] for q in range(case["n"]) if q != case["rank"]]}
