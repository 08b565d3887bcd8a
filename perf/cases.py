"""Performance cases of the SpMM / SDDMM library: the calls a user's program makes, over the range it makes them in.

A case is a dict of plain values:
  op      step     SpMM and SDDMM on a plan that is kept, into outputs that are kept (the benchmark's step)
          spmm     SpMM alone, output allocated by the call (inference of a graph network's aggregation)
          head     an attention head: SDDMM -> edge softmax -> new values -> SpMM (K = N)
          plan     the same step on a matrix seen for the first time: plan on the GPU, then SpMM and SDDMM
          gcn      a training layer with fixed edge weights: SpMM forward, gradient of the features
          agnn     a training layer with attention: SDDMM -> edge softmax -> SpMM forward, gradient of the features (K = N)
  kind    rmat       R-MAT power-law graph, symmetrised (`degree` directed samples per row before that), unit values
          community  diagonal blocks of 64 x 64 at density 0.3 and two columns per row outside them, values U(-1, 1)
          zipf       rows with shifted Zipf degrees (mean 50, up to 1e5), uniform columns, unit values
          uniform    `degree` uniform columns per row, values U(-1, 1)
  rows, cols, degree   size of the matrix (cols = rows but for `uniform`)
  dtype   storage type of values and dense operands;  N, K   feature widths of SpMM and SDDMM
  tuned   options from the tuner's table (what the benchmark uses) or the library's defaults

Everything is drawn on the GPU from the seed: another seed is another matrix (with the same number of nonzeros) and other
operands.
"""
from __future__ import annotations

import math
import os

import numpy as np
import torch

from paper_2506_22714_amd import autograd as ag
from paper_2506_22714_amd import binding as lb

TUNED = os.path.join(os.path.dirname(os.path.abspath(lb.__file__)), "tuned_gfx950.json")
DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
BLOCK, DENSITY, OFF_BLOCK = 64, 0.3, 2
ZIPF_EXPONENT, ZIPF_SHIFT, ZIPF_MAX = 2.1, 8.2003, 100_000


def _case(name, op, kind, rows, dtype, N, K, cols=0, degree=0, tuned=True):
    return dict(name=name, op=op, kind=kind, rows=rows, cols=cols or rows, degree=degree, dtype=dtype, N=N, K=K, tuned=tuned)


def listed():
    return [
        # a matrix that fits in the caches, smallest widths: launch and call latency
        _case("tiny_step", "step", "uniform", 2048, "f16", 32, 32, degree=16),
        # training on a small graph: some twenty short calls a layer
        _case("small_graph_training", "agnn", "rmat", 4096, "f16", 32, 32, degree=16, tuned=False),
        # a sampled neighbourhood of mini-batch training: a ragged, non-square matrix that is new in every step
        _case("minibatch_plan", "plan", "uniform", 8191, "bf16", 96, 64, cols=50021, degree=10, tuned=False),
        # the benchmark's step: power-law graph, wide SpMM and narrow SDDMM
        _case("powerlaw_step", "step", "rmat", 1 << 17, "f16", 128, 32, degree=16),
        # aggregation of a wide hidden layer over a larger graph, ragged row count
        _case("powerlaw_wide", "spmm", "rmat", 200003, "bf16", 256, 32, degree=16),
        # block-structured matrix whose nonzeros mostly run on the matrix cores
        _case("community_step", "step", "community", 1 << 20, "f16", 128, 32),
        # the same structure in fp32, ragged row count, a width that is cut into two pieces, widest SDDMM
        _case("community_f32", "step", "community", 300017, "f32", 96, 128),
        # the largest: 120 M nonzeros with no structure, operands larger than any L2
        _case("irregular_step", "step", "zipf", 2_400_000, "f16", 32, 32),
        # graph attention inference on a large power-law graph
        _case("gat_head", "head", "rmat", 1 << 20, "f16", 64, 64, degree=32),
        # the same graph seen for the first time: preprocessing on the GPU and one step
        _case("gat_plan", "plan", "rmat", 1 << 20, "f16", 64, 64, degree=32),
        # attention training on a large graph: forward and backward
        _case("attention_training", "agnn", "rmat", 500009, "bf16", 64, 64, degree=16, tuned=False),
        # convolution training on an irregular graph: forward and backward, wide features
        _case("convolution_training", "gcn", "zipf", 300007, "f16", 128, 32, tuned=False),
    ]


def draw(rng):
    op = rng.choice(["step", "step", "spmm", "head", "plan", "gcn", "agnn"])
    kind = rng.choice(["rmat", "rmat", "community", "zipf", "uniform"])
    dtype = rng.choice(["f16", "f16", "bf16", "f32"])
    K = rng.choice([32, 64, 128])
    # whole widths of hidden layers most of the time, any legal multiple otherwise
    unit = 16 if dtype == "f32" else 32
    N = K if op in ("head", "agnn") else rng.choice([32, 64, 128, 256, 512, unit * rng.randint(1, 512 // unit)])
    degree = rng.randint(4, 48)
    per_row = {"rmat": 1.8 * degree, "community": 21.2, "zipf": 50.0, "uniform": degree}[kind]
    # nonzeros log-uniform from a few ten thousand to 20 million; dense operands of at most 256 M values
    nnz = math.exp(rng.uniform(math.log(3e4), math.log(2e7)))
    rows = max(300, min(int(nnz / per_row), (1 << 28) // max(N, K))) | 1
    cols = rows
    if kind == "uniform":
        cols = max(256, min(int(rows * math.exp(rng.uniform(math.log(0.25), math.log(8.0)))), (1 << 28) // max(N, K)))
        degree = min(degree, cols // 8)
    c = _case("", op, kind, rows, dtype, N, K, cols=cols, degree=degree if kind in ("rmat", "uniform") else 0, tuned=rng.random() < 0.5)
    del c["name"]
    return c


# ---- inputs -----------------------------------------------------------------------------------------------------------
def _samples(case, gen, share):
    """Keys row * cols + col, duplicates among them: about `share` times what the kind of matrix holds."""
    M, Kc, kind = case["rows"], case["cols"], case["kind"]
    rand = lambda n: torch.rand(n, device="cuda", generator=gen)  # noqa: E731
    randint = lambda hi, n: torch.randint(hi, (n,), device="cuda", generator=gen)  # noqa: E731
    if kind == "rmat":
        a, b, c = 0.57, 0.19, 0.19
        scale, ns = max(1, (M - 1).bit_length()), int(M * case["degree"] * share) + 1
        src = torch.zeros(ns, dtype=torch.int64, device="cuda")
        dst = torch.zeros_like(src)
        for _ in range(scale):
            u = rand(ns)
            src = (src << 1) | (u >= a + b)
            dst = (dst << 1) | (((u >= a) & (u < a + b)) | (u >= a + b + c))
        if M != 1 << scale:  # node ids squeezed onto a row count that is no power of two
            src, dst = src * M >> scale, dst * M >> scale
        return torch.cat([src * M + dst, dst * M + src])
    if kind == "community":
        if share < 1.0:  # single places of the diagonal blocks
            rows = randint(M, int(M * BLOCK * DENSITY * share) + 1)
            start = rows // BLOCK * BLOCK
            return rows * Kc + start + (rand(rows.numel()) * (Kc - start).clamp(max=BLOCK)).long()
        parts = []
        nb = -(-M // BLOCK)
        for b0 in range(0, nb, 4096):
            n = min(4096, nb - b0)
            bi, ri, ci = torch.nonzero(rand(n * BLOCK * BLOCK).view(n, BLOCK, BLOCK) < DENSITY, as_tuple=True)
            r, c = (bi + b0) * BLOCK + ri, (bi + b0) * BLOCK + ci
            inside = (r < M) & (c < Kc)  # the last block ends at the matrix's edge
            parts.append(r[inside] * Kc + c[inside])
        rows = torch.arange(M, device="cuda").repeat_interleave(OFF_BLOCK)
        return torch.cat(parts + [rows * Kc + randint(Kc, rows.numel())])
    if kind == "zipf":
        d = torch.arange(1, min(ZIPF_MAX, Kc) + 1, dtype=torch.float64, device="cuda")
        cdf = torch.cumsum((d + ZIPF_SHIFT) ** -ZIPF_EXPONENT, 0)
        n = int(M * share) + 1
        deg = torch.searchsorted(cdf / cdf[-1], rand(n).double()).clamp_(max=d.numel() - 1) + 1
        rows = (torch.arange(n, device="cuda") if share >= 1.0 else randint(M, n)).clamp_(max=M - 1).repeat_interleave(deg)
    else:
        rows = torch.arange(M, device="cuda").repeat_interleave(case["degree"]) if share >= 1.0 else randint(M, int(M * case["degree"] * share) + 1)
    return rows * Kc + randint(Kc, rows.numel())


def _pattern(case, gen):
    """Sorted unique keys row * cols + col on the GPU, as many as _nnz says: samples until there are enough, the surplus
    dropped at random."""
    want = _nnz(case)
    keys = torch.unique(_samples(case, gen, 1.0))
    while keys.numel() < want:
        keys = torch.unique(torch.cat([keys, _samples(case, gen, 0.05)]))
    if keys.numel() > want:
        keep = torch.ones(keys.numel(), dtype=torch.bool, device="cuda")
        keep[torch.randperm(keys.numel(), device="cuda", generator=gen)[want:]] = False
        keys = keys[keep]
    return keys


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    M, Kc, N, K, op = case["rows"], case["cols"], case["N"], case["K"], case["op"]
    dtype = DTYPES[case["dtype"]]
    keys = _pattern(case, gen)
    rows, col = keys // Kc, (keys % Kc).int()
    nnz = keys.numel()
    counts = torch.bincount(rows, minlength=M)
    rowptr = torch.zeros(M + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.cumsum(counts, 0)
    del keys
    graph = case["kind"] in ("rmat", "zipf")
    if op == "gcn" and M == Kc:  # the symmetric normalisation 1 / sqrt(d_i d_j)
        d = counts.clamp(min=1).float()
        val = (d[rows] * d[col.long()]).rsqrt().to(dtype)
    elif graph or op == "agnn":
        val = torch.ones(nnz, dtype=dtype, device="cuda")
    else:
        val = ((torch.rand(nnz, device="cuda", generator=gen) * 2 - 1) * 0.999 + 0.001).to(dtype)
    del rows
    dense = lambda r, c: torch.randn(r, c, device="cuda", generator=gen).to(dtype)  # noqa: E731
    s = dict(op=op, M=M, Kc=Kc, N=N, K=K, val=val, scale=1.0 / math.sqrt(K), nnz=nnz)
    s["opts"] = dict(tuned=TUNED, N=N, K=K) if case["tuned"] else {}
    if op in ("gcn", "agnn"):
        s["matrix"] = ag.SparseMatrix(M, Kc, rowptr, col, dtype=dtype)
        if op == "gcn":
            s["Z"] = dense(Kc, N).requires_grad_()
        else:
            s["Q"], s["Z"] = dense(M, K).requires_grad_(), dense(Kc, N).requires_grad_()
        s["dC"] = torch.randn(M, N, device="cuda", generator=gen)
        return s
    s["B"] = dense(Kc, N)
    if op != "spmm":
        s["X"], s["Y"] = dense(M, K), s["B"] if op == "head" else dense(Kc, K)
    if op == "plan":
        s["rowptr"], s["col"] = rowptr, col
        return s
    s["plan"] = lb.Plan.from_device_csr(M, Kc, rowptr, col, val, resident=True, keep_host_copy=False, **s["opts"])
    if op in ("step", "head"):
        s["C"] = torch.empty(M, N, dtype=torch.float32, device="cuda")
        s["out"] = torch.empty(nnz, dtype=torch.float32, device="cuda")
    if op == "head":
        s["alpha"] = torch.empty(nnz, dtype=dtype, device="cuda")
    return s


def run(s):
    op = s["op"]
    if op == "step":
        return s["plan"].spmm(s["B"], out=s["C"]), s["plan"].sddmm(s["X"], s["Y"], out=s["out"])
    if op == "spmm":
        return s["plan"].spmm(s["B"])
    if op == "head":
        p = s["plan"]
        scores = p.sddmm(s["X"], s["Y"], out=s["out"])
        alpha = p.edge_softmax(scores, s["scale"], out=s["alpha"])
        p.set_values(alpha, lb.OP_SPMM)
        return scores, alpha, p.spmm(s["B"], out=s["C"])
    if op == "plan":
        p = lb.Plan.from_device_csr(s["M"], s["Kc"], s["rowptr"], s["col"], s["val"], resident=True, keep_host_copy=False, **s["opts"])
        C, out = p.spmm(s["B"]), p.sddmm(s["X"], s["Y"])
        p.close()
        return C, out
    if op == "gcn":
        C = ag.spmm(s["matrix"], s["val"], s["Z"])
        (dZ,) = torch.autograd.grad(C, (s["Z"],), s["dC"])
        return C.detach(), dZ
    scores = ag.sddmm(s["matrix"], s["val"], s["Q"], s["Z"])
    alpha = ag.edge_softmax(s["matrix"], scores, s["scale"])
    C = ag.spmm(s["matrix"], alpha, s["Z"])
    dQ, dZ = torch.autograd.grad(C, (s["Q"], s["Z"]), s["dC"])
    return C.detach(), alpha.detach(), dQ, dZ


# ---- what a pass cannot do without ------------------------------------------------------------------------------------
def _nnz(case):
    M, Kc = case["rows"], case["cols"]
    if case["kind"] == "rmat":  # both directions, a tenth of them merged
        return int(1.78 * M * case["degree"])
    if case["kind"] == "community":
        return int(M * (BLOCK * DENSITY + OFF_BLOCK) * 0.99)
    if case["kind"] == "zipf":
        d = np.arange(1, min(ZIPF_MAX, Kc) + 1, dtype=np.float64)
        p = (d + ZIPF_SHIFT) ** -ZIPF_EXPONENT
        return int(M * (d * p).sum() / p.sum() * 0.97)
    return M * case["degree"]


def work(case):
    M, Kc, N, K, op = case["rows"], case["cols"], case["N"], case["K"], case["op"]
    es, nnz = (4 if case["dtype"] == "f32" else 2), _nnz(case)
    csr = nnz * (4 + es) + 4 * (M + 1)                       # columns, values, row pointers, read once
    used = 0.7 if case["kind"] == "rmat" else 1.0            # rows of an operand that some nonzero refers to
    spmm = csr + used * Kc * N * es + M * N * 4
    sddmm = csr + used * (M + Kc) * K * es + nnz * 4
    softmax = nnz * (4 + es) + 4 * (M + 1)
    values = nnz * 2 * es                                    # read in one order, written in another
    f_spmm, f_sddmm = 2.0 * nnz * N, 2.0 * nnz * K
    if op == "spmm":
        return {"bytes": spmm, "flops": f_spmm}
    if op == "step":
        return {"bytes": spmm + sddmm, "flops": f_spmm + f_sddmm}
    if op == "head":
        return {"bytes": sddmm + softmax + values + spmm, "flops": f_spmm + f_sddmm}
    if op == "plan":                                         # the matrix once, each operator's form of it once, the step
        return {"bytes": csr + 2 * nnz * (4 + es) + spmm + sddmm, "flops": f_spmm + f_sddmm}
    spmm_t = csr + M * N * (4 + es) + Kc * N * 2 * es        # gradient rounded to the operand type, result too
    if op == "gcn":
        return {"bytes": 2 * values + spmm + spmm_t, "flops": 2 * f_spmm}
    forward = values + sddmm + softmax + values + spmm
    softmax_b = nnz * (es + 8) + 4 * (M + 1)
    # dC -> dalpha (SDDMM) and dZ (transposed SpMM); dalpha -> dscores; dscores -> dQ (SpMM) and dZ (transposed SpMM)
    backward = sddmm + values + spmm_t + softmax_b + nnz * (4 + 2 * es) + values + spmm + values + spmm_t
    return {"bytes": forward + backward, "flops": 4 * f_spmm + 2 * f_sddmm}


def tolerance(case):
    """About four times what the same cases differ by with their sums in another order (scalar-only plans with other segment
    lengths against hybrid ones): fp32 sums 2.5e-7 (worst value 7e-5); where results or intermediate coefficients are rounded
    to 16 bits a sum that moved rounds the other way now and then: f16 2.3e-5 (worst 1.3e-3), bf16 4.8e-5 (worst 2.7e-2)."""
    if case["op"] in ("step", "spmm", "plan") or case["dtype"] == "f32":
        return {"rel": 1e-6, "max": 3e-4}
    return {"rel": 1e-4, "max": 5e-3} if case["dtype"] == "f16" else {"rel": 2e-4, "max": 0.1}
