"""Performance cases of the GEMM library: what a program calls it for, over the
range of sizes, types and options that it takes.

A case is a dict of plain values; "kind" names the entry point:

  dense    one C <- alpha*A*B + beta*C in binary32 ("f32"), or FP32-accurate
           split precision with three or six products ("split3", "split6");
           "trans" other than "NN" goes through gemm_ex
  skinny   a split-precision product of few rows, in one pass, or split over k
           with a workspace that the caller keeps ("ws") or without one
           ("noalloc")
  fp8      scaled FP8, quantisation of both operands included, or from the
           codes of an earlier quantisation ("pre")
  f64      one binary64 product
  batch    a batch of equally shaped small products at fixed strides
  grouped  a batch of uneven products in one launch: a graph captured once and
           replayed, or the direct call
  serve    a burst of requests on host buffers through the serving loop
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1902_10345_amd as mm

_PATH = {"f32": mm.PATH_F32, "split3": mm.PATH_3XBF16, "split6": mm.PATH_3XBF16}


def listed():
    return [
        # the smallest call of the benchmark: launch and latency
        _dense("f32_256", "f32", 256, 256, 256, beta=0.0),
        # the plain binary32 product at the benchmark's rectangular size
        _dense("f32_8192x2048x4096", "f32", 8192, 2048, 4096, beta=0.5),
        # the headline: FP32-accurate split precision, 4096^3
        _dense("split3_4096", "split3", 4096, 4096, 4096, beta=0.5),
        # the paper's own matrix multiplication, C = A*B at 2048^3
        _dense("split3_2048", "split3", 2048, 2048, 2048, beta=0.0),
        # a ragged product with a transposed operand (the A^T B of a backward
        # pass), six products, accumulated into C
        _dense("split6_TN_1531x1111x2047", "split6", 1531, 1111, 2047, beta=1.0, trans="TN"),
        # few rows against a large matrix: a small batch at a dense layer
        dict(name="skinny_64x4096x4096", kind="skinny", m=64, n=4096, k=4096, beta=0.5,
             n_products=3, split="one"),
        # scaled FP8 with the quantisation of both operands
        dict(name="fp8_4096", kind="fp8", m=4096, n=4096, k=4096, beta=0.5, pre=False),
        # binary64, sizes that no tile divides
        dict(name="f64_1999x1501x1003", kind="f64", m=1999, n=1501, k=1003, beta=0.5),
        # the paper's batched small product (binary64, 1.92 GFLOP of 32^3)
        dict(name="batch_f64_32_x29297", kind="batch", dtype="f64", m=32, n=32, k=32, beta=0.0,
             batch=29297),
        # a batch of medium, ragged problems in binary32
        dict(name="batch_f32_100x72x90_x2000", kind="batch", dtype="f32", m=100, n=72, k=90,
             beta=0.0, batch=2000),
        # the benchmark's grouped batch: 512 problems, sizes log-uniform in
        # [32, 1024], replayed as a graph
        dict(name="grouped_512", kind="grouped", count=512, lo=32, hi=1024, multiple=16,
             sizes_seed=5, graph=True),
        # a burst of ragged requests, sizes log-uniform in [64, 2048]
        dict(name="serve_32", kind="serve", count=32, lo=64, hi=2048, sizes_seed=6),
    ]


def _dense(name, path, m, n, k, beta, trans="NN"):
    return dict(name=name, kind="dense", path=path, m=m, n=n, k=k, beta=beta, trans=trans)


def _size(rng, lo, hi):
    """Log-uniform in [lo, hi]; half of the draws on a multiple of 16."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    if rng.random() < 0.5 and v >= 16:
        v = round(v / 16) * 16
    return int(min(max(round(v), lo), hi))


def draw(rng):
    kind = rng.choice(["dense"] * 6 + ["skinny"] * 2 + ["fp8"] * 2 + ["f64"] * 2 + ["batch"] * 4 +
                      ["grouped"] * 2 + ["serve"])
    beta = rng.choice([0.0, 0.5, 1.0])
    if kind == "dense":
        m, n, k = (_size(rng, 32, 4096) for _ in range(3))
        return dict(kind=kind, path=rng.choice(["f32", "split3", "split3", "split6"]), m=m, n=n,
                    k=k, beta=beta, trans=rng.choice(["NN", "NN", "NN", "NT", "TN", "TT"]))
    if kind == "skinny":
        return dict(kind=kind, m=_size(rng, 1, 128), n=_size(rng, 1024, 8192),
                    k=_size(rng, 1024, 8192), beta=beta, n_products=rng.choice([3, 3, 6]),
                    split=rng.choice(["one", "one", "ws", "noalloc"]))
    if kind == "fp8":
        return dict(kind=kind, m=_size(rng, 64, 4096), n=_size(rng, 64, 4096),
                    k=_size(rng, 64, 4096), beta=beta, pre=rng.random() < 0.5)
    if kind == "f64":
        return dict(kind=kind, m=_size(rng, 32, 2048), n=_size(rng, 32, 2048),
                    k=_size(rng, 32, 2048), beta=beta)
    if kind == "batch":
        dtype = rng.choice(["f64", "f32", "split3", "split6"])
        m, n, k = (_size(rng, 4, 160) for _ in range(3))
        # enough problems for about 16 to 128 MB of operands, 50000 at most
        each = (8 if dtype == "f64" else 4) * (m * k + k * n + m * n)
        total = math.exp(rng.uniform(math.log(16e6), math.log(128e6)))
        return dict(kind=kind, dtype=dtype, m=m, n=n, k=k, beta=beta,
                    batch=int(min(50000, max(2, total / each))))
    if kind == "grouped":
        return dict(kind=kind, count=_size(rng, 32, 512), lo=32, hi=1024,
                    multiple=rng.choice([1, 16]), sizes_seed=rng.randrange(1 << 20),
                    graph=rng.random() < 0.5)
    return dict(kind=kind, count=_size(rng, 8, 32), lo=64, hi=2048,
                sizes_seed=rng.randrange(1 << 20))


def _sizes(case):
    """count (M, N, K), log-uniform in [lo, hi], on the case's multiple."""
    g = np.random.default_rng(case["sizes_seed"])
    mult = case.get("multiple", 1)
    raw = np.exp(g.uniform(math.log(case["lo"]), math.log(case["hi"]), size=(case["count"], 3)))
    r = np.clip(np.rint(raw / mult) * mult, case["lo"], case["hi"]).astype(np.int64)
    return [(int(a), int(b), int(c)) for a, b, c in r]


def work(case):
    kind = case["kind"]
    if kind in ("grouped", "serve"):
        s = _sizes(case)
        return {"bytes": sum(4.0 * (m * k + k * n + m * n) for m, n, k in s),
                "flops": sum(2.0 * m * n * k for m, n, k in s)}
    m, n, k, b = case["m"], case["n"], case["k"], case.get("batch", 1)
    c = (2 if case["beta"] else 1) * m * n
    if kind == "fp8" and case["pre"]:
        return {"bytes": 1.0 * (m * k + k * n) + 4.0 * (m + n + c), "flops": 2.0 * m * n * k}
    each = 8.0 if kind == "f64" or case.get("dtype") == "f64" else 4.0
    return {"bytes": b * each * (m * k + k * n + c), "flops": b * 2.0 * m * n * k}


class _Inputs:
    """Seeded device tensors: uniform [-1, 1), the values of the benchmark's
    products, or N(0, 1) for the FP8 path."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def uniform(self, *shape, dtype=torch.float32):
        t = torch.rand(*shape, generator=self.g, device="cuda", dtype=dtype)
        return t.mul_(2.0).sub_(1.0)

    def normal(self, *shape):
        return torch.randn(*shape, generator=self.g, device="cuda", dtype=torch.float32)


class _Server:
    """A server and its arena, closed with the state that holds it."""

    def __init__(self, arena_bytes, slots):
        self.arena = torch.empty(arena_bytes, dtype=torch.uint8, device="cuda")
        self.handle = mm.server_create(self.arena, arena_bytes, slots, mm.PATH_3XBF16, 4)

    def __del__(self):
        if getattr(self, "handle", None):
            mm.server_destroy(self.handle)


class _Graph:
    """A captured grouped launch, destroyed with the state that holds it."""

    def __init__(self, arr, count, ws):
        self.handle = mm.grouped_graph_create(arr, count, mm.PATH_3XBF16, None, ws, ws.numel())

    def __del__(self):
        if getattr(self, "handle", None):
            torch.cuda.synchronize()
            mm.grouped_graph_destroy(self.handle)


def _flat_outputs(sizes, dtype):
    """One buffer for the outputs of a grouped batch, each at a 256-byte
    boundary, and their views in it."""
    at, end = [], 0
    for m, n, _ in sizes:
        at.append(end)
        end += (m * n + 63) // 64 * 64
    flat = torch.zeros(end, dtype=dtype, device="cuda")
    return flat, [flat[o:o + m * n].view(m, n) for o, (m, n, _) in zip(at, sizes)]


def _operands(case, seed):
    """Operands as stored and C of one product (or of a batch of them)."""
    g, kind = _Inputs(seed), case["kind"]
    m, n, k, beta = case["m"], case["n"], case["k"], case["beta"]
    dtype = torch.float64 if kind == "f64" or case.get("dtype") == "f64" else torch.float32
    lead = (case["batch"],) if kind == "batch" else ()
    trans = case.get("trans", "NN")
    sa = (k, m) if trans[0] == "T" else (m, k)
    sb = (n, k) if trans[1] == "T" else (k, n)
    if kind == "fp8":
        a, b = g.normal(*sa), g.normal(*sb)
    else:
        a, b = g.uniform(*lead, *sa, dtype=dtype), g.uniform(*lead, *sb, dtype=dtype)
    c = (g.uniform(*lead, m, n, dtype=dtype) if beta
         else torch.empty(*lead, m, n, dtype=dtype, device="cuda"))
    return a, b, c


def prepare(case, seed):
    kind = case["kind"]
    state = dict(case=case)
    if kind in ("grouped", "serve"):
        sizes = _sizes(case)
        g = _Inputs(seed)
        ops = [(m, n, k, g.uniform(m, k), g.uniform(k, n)) for m, n, k in sizes]
        if kind == "serve":
            state["reqs"] = [(m, n, k, a.cpu().pin_memory(), b.cpu().pin_memory(),
                              torch.empty((m, n), pin_memory=True)) for m, n, k, a, b in ops]
            need = sum(4 * (m * k + k * n + m * n) + 1024 for m, n, k in sizes)
            state["server"] = _Server(need + (16 << 20), 64)
            return state
        state["flat"], state["out"] = _flat_outputs(sizes, torch.float32)
        state["ops"] = ops
        state["arr"] = mm.problem_array([(m, n, k, a, k, b, n, c, n, 1.0, 0.0)
                                         for (m, n, k, a, b), c in zip(ops, state["out"])])
        state["ws"] = torch.empty(mm.grouped_gemm_workspace_bytes(len(sizes)), dtype=torch.uint8,
                                  device="cuda")
        if case["graph"]:
            state["graph"] = _Graph(state["arr"], len(sizes), state["ws"])
        return state
    state["a"], state["b"], state["c"] = _operands(case, seed)
    m, n, k = case["m"], case["n"], case["k"]
    if kind == "skinny" and case["split"] == "ws":
        nbytes = mm.gemm_splitk_workspace_bytes(m, n, k, 0)
        state["ws"] = torch.empty(max(nbytes, 256), dtype=torch.uint8, device="cuda")
    if kind == "fp8":
        nbytes = mm.gemm_fp8_workspace_bytes(m, n, k)
        state["ws"] = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        if case["pre"]:
            mm.fp8_quantize(m, n, k, state["a"], k, state["b"], n, state["ws"], nbytes)
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "grouped":
        if case["graph"]:
            mm.grouped_graph_launch(state["graph"].handle)
        else:
            mm.grouped_gemm(state["arr"], case["count"], mm.PATH_3XBF16, None, state["ws"],
                            state["ws"].numel())
        return state["flat"]
    if kind == "serve":
        h = state["server"].handle
        tickets = [mm.server_submit(h, m, n, k, 1.0, a, b, 0.0, None, c)
                   for m, n, k, a, b, c in state["reqs"]]
        mm.server_drain(h, 60.0)
        for t in tickets:
            mm.server_poll(h, t)
        return [r[5] for r in state["reqs"]]
    a, b, c = state["a"], state["b"], state["c"]
    m, n, k, beta = case["m"], case["n"], case["k"], case["beta"]
    alpha = 1.5 if beta == 0.5 else 1.0
    if kind == "dense":
        path, trans = case["path"], case["trans"]
        if trans != "NN":
            ta, tb = trans[0] == "T", trans[1] == "T"
            mm.gemm_ex(mm.ROW_MAJOR, mm.TRANS if ta else mm.NO_TRANS,
                       mm.TRANS if tb else mm.NO_TRANS, m, n, k, alpha, a, m if ta else k, b,
                       k if tb else n, beta, c, n, _PATH[path], 6 if path == "split6" else 3)
        elif path == "f32":
            mm.gemm_f32(m, n, k, alpha, a, k, b, n, beta, c, n)
        else:
            mm.gemm_f32_3xbf16(m, n, k, alpha, a, k, b, n, beta, c, n, int(path[-1]))
    elif kind == "skinny":
        if case["split"] == "ws":
            mm.gemm_f32_3xbf16_splitk(m, n, k, alpha, a, k, b, n, beta, c, n, case["n_products"],
                                      0, state["ws"], state["ws"].numel())
        elif case["split"] == "noalloc":
            mm.gemm_f32_3xbf16_splitk_noalloc(m, n, k, alpha, a, k, b, n, beta, c, n,
                                              case["n_products"], 0)
        else:
            mm.gemm_f32_3xbf16(m, n, k, alpha, a, k, b, n, beta, c, n, case["n_products"])
    elif kind == "fp8":
        ws = state["ws"]
        if case["pre"]:
            mm.gemm_fp8_prequantized(m, n, k, alpha, ws, ws.numel(), beta, c, n)
        else:
            mm.gemm_fp8_scaled(m, n, k, alpha, a, k, b, n, beta, c, n, ws, ws.numel())
    elif kind == "f64":
        mm.gemm_f64(m, n, k, alpha, a, k, b, n, beta, c, n)
    elif case["dtype"] == "f64":
        mm.gemm_f64_strided_batched(m, n, k, alpha, a, k, m * k, b, n, k * n, beta, c, n, m * n,
                                    case["batch"])
    else:
        mm.gemm_strided_batched(_PATH[case["dtype"]], m, n, k, alpha, a, k, m * k, b, n, k * n,
                                beta, c, n, m * n, case["batch"],
                                6 if case["dtype"] == "split6" else 3)
    return c


def _dequantised(x, dim):
    """The values that the E4M3 codes and binary32 scales along `dim` stand for."""
    amax = x.abs().amax(dim=dim, keepdim=True)
    # a tensor divisor: division by a Python number multiplies by its reciprocal
    s = torch.where(amax == 0, torch.ones_like(amax), amax / torch.full_like(amax, 448.0))
    q = (x / s).clamp(-448.0, 448.0).to(torch.float8_e4m3fn)
    return q.to(torch.float64) * s.to(torch.float64)


def exact(case, seed):
    """The outputs of run() in 64 bits: for FP8 the exact product of the
    quantised operands."""
    kind = case["kind"]
    if kind in ("grouped", "serve"):
        g, sizes = _Inputs(seed), _sizes(case)
        flat, out = _flat_outputs(sizes, torch.float64)
        for (m, n, k), c in zip(sizes, out):
            a, b = g.uniform(m, k), g.uniform(k, n)
            c.copy_(torch.matmul(a.double(), b.double()))
        return flat if kind == "grouped" else out
    a, b, c = _operands(case, seed)
    trans = case.get("trans", "NN")
    beta = case["beta"]
    alpha = 1.5 if beta == 0.5 else 1.0
    if kind == "fp8":
        a, b = _dequantised(a, 1), _dequantised(b, 0)
    a = a.transpose(-1, -2) if trans[0] == "T" else a
    b = b.transpose(-1, -2) if trans[1] == "T" else b
    r = alpha * torch.matmul(a.double().contiguous(), b.double().contiguous())
    return r + beta * c.double() if beta else r
