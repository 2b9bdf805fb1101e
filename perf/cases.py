"""The calls this library is timed on: what its users have it do, over the range of sizes they do it at.

A case is a dict of plain values.  ``kind`` says which program it stands for, the other entries its sizes:

* ``gemm``    one kept plan, one call (hgemm_plan + hgemm_run): aligned problems from the small corner of the
              {64 ... 16384}^3 shape grid to its large one, in both layouts of B, packed or inside wider buffers;
* ``batch``   the paper's offline mode: back-to-back calls of one plan over several operand sets (hgemm_run_many),
              where a call takes no longer than its launch;
* ``layer``   the projections of one transformer layer applied to ``m`` tokens (attention square, attention output is
              the same shape; up, down and fused gate), one plan each, kept with the weights: decoding at a few rows, prefill
              at hundreds;
* ``ragged``  a problem whose dimensions nobody rounded (odd sizes, a vocabulary's output head), one kept plan;
* ``static``  plan and run in one call that allocates nothing (hgemm_run_static), as a serving loop does it, with
              operands that are slices of wider buffers;
* ``oneshot`` the convenience call hgemm(a, b) on two tensors.
"""
from __future__ import annotations

import torch

import paper_2512_02551_amd as hg

# widths of the transformer layer whose projections the layer cases run: model width and feed-forward widths
WIDTH, UP, FUSED = 4096, 11008, 14336


def listed():
    return [
        # the smallest calls: 256^3, eight of them enqueued back to back
        {"name": "batch 8 x 256^3", "kind": "batch", "m": 256, "n": 256, "k": 256, "count": 8, "tn": False},
        # the square sweep: small, ordinary, large (column-major B, as the weights of a linear layer lie)
        {"name": "square 1024", "kind": "gemm", "m": 1024, "n": 1024, "k": 1024, "tn": False, "gap": 0},
        {"name": "square 4096", "kind": "gemm", "m": 4096, "n": 4096, "k": 4096, "tn": False, "gap": 0},
        {"name": "square 8192 tn", "kind": "gemm", "m": 8192, "n": 8192, "k": 8192, "tn": True, "gap": 0},
        # the largest problem of the benchmark's configurations
        {"name": "16384 x 16384 x 8192", "kind": "gemm", "m": 16384, "n": 16384, "k": 8192, "tn": False, "gap": 0},
        # one layer's projections: one token, a small batch of requests, a prompt
        {"name": "layer 1 token", "kind": "layer", "m": 1, "width": WIDTH, "up": UP, "fused": FUSED, "tn": False},
        {"name": "layer 16 tokens tn", "kind": "layer", "m": 16, "width": WIDTH, "up": UP, "fused": FUSED, "tn": True},
        {"name": "layer 512 tokens", "kind": "layer", "m": 512, "width": WIDTH, "up": UP, "fused": FUSED, "tn": False},
        # nothing divides by anything
        {"name": "ragged 1000x1001x1003", "kind": "ragged", "m": 1000, "n": 1001, "k": 1003, "tn": False},
        # the output head over a vocabulary of odd size
        {"name": "head 16x50257x4096", "kind": "ragged", "m": 16, "n": 50257, "k": 4096, "tn": True},
        # a serving loop's call on a third of a fused buffer, a shape that nobody tuned
        {"name": "static 320x3072x768", "kind": "static", "m": 320, "n": 3072, "k": 768, "tn": False, "gap": 1536},
        # the first call of the README on a shape that nobody tuned
        {"name": "oneshot 1536^3", "kind": "oneshot", "m": 1536, "n": 1536, "k": 1536, "tn": False},
    ]


def _size(rng, lo, hi, step=1):
    """A size from lo to hi, spread over its logarithm, a multiple of step."""
    v = lo * (hi / lo) ** rng.random()
    return int(min(max(round(v / step) * step, lo), hi))


def draw(rng):
    kind = rng.choice(["gemm", "gemm", "gemm", "batch", "layer", "layer", "ragged", "ragged", "static", "oneshot"])
    tn = rng.random() < 0.5
    if kind == "gemm":
        while True:
            m, n, k = _size(rng, 64, 16384), _size(rng, 64, 16384, 8), _size(rng, 64, 16384, 8)
            if m * n * k <= 1 << 41:
                return {"kind": kind, "m": m, "n": n, "k": k, "tn": tn, "gap": rng.choice([0, 0, 8 * rng.randint(1, 64)])}
    if kind == "batch":
        return {"kind": kind, "m": _size(rng, 16, 512), "n": _size(rng, 64, 512, 8), "k": _size(rng, 64, 1024, 8), "count": rng.randint(4, 16), "tn": tn}
    if kind == "layer":
        width = _size(rng, 1024, 8192, 128)
        up = int(width * rng.uniform(2.5, 4.0)) // 128 * 128
        return {"kind": kind, "m": _size(rng, 1, 768), "width": width, "up": up, "fused": up + width, "tn": tn}
    if kind == "ragged":
        if rng.random() < 0.5:      # the output head of a model: few rows, a long odd side
            return {"kind": kind, "m": _size(rng, 1, 64), "n": _size(rng, 8000, 64000) | 1, "k": _size(rng, 512, 8192, 8), "tn": tn}
        return {"kind": kind, "m": _size(rng, 65, 4200), "n": _size(rng, 65, 4200) | 1, "k": _size(rng, 129, 4200) | 1, "tn": tn}
    if kind == "static":
        return {"kind": kind, "m": _size(rng, 1, 1024), "n": _size(rng, 64, 4096, 8), "k": _size(rng, 64, 1024, 8), "tn": tn,
                "gap": 8 * rng.randint(0, 256)}
    return {"kind": kind, "m": _size(rng, 64, 4096), "n": _size(rng, 64, 4096, 8), "k": _size(rng, 64, 4096, 8), "tn": tn}


def _products(case):
    """The (M, N, K) of the products of one pass."""
    m = case["m"]
    if case["kind"] == "layer":
        w, u, f = case["width"], case["up"], case["fused"]
        return [(m, w, w), (m, u, w), (m, w, u), (m, f, w)]
    return [(m, case["n"], case["k"])] * (case["count"] if case["kind"] == "batch" else 1)


def _inputs(case, seed):
    """The operands of every product: activations N(0, 1) and weights N(0, 0.02^2) for a layer and a head, N(0, 1) / sqrt(K)
    for the squares and batches, uniform in [-1, 1) otherwise.  B is N x K where it is column-major.  A gap puts A into a
    buffer whose rows are that much longer."""
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)
    out = []
    for m, n, k in _products(case):
        bshape = (n, k) if case["tn"] else (k, n)
        lda = k + case.get("gap", 0)
        if case["kind"] == "layer" or (case["kind"] == "ragged" and m <= 64):
            a = torch.randn((m, lda), generator=g, device="cuda").half()
            b = torch.randn(bshape, generator=g, device="cuda").mul_(0.02).half()
        elif case["kind"] == "batch" or m == n == k:
            a = torch.randn((m, lda), generator=g, device="cuda").mul_(k ** -0.5).half()
            b = torch.randn(bshape, generator=g, device="cuda").mul_(k ** -0.5).half()
        else:
            a = torch.rand((m, lda), generator=g, device="cuda").mul_(2.0).sub_(1.0).half()
            b = torch.rand(bshape, generator=g, device="cuda").mul_(2.0).sub_(1.0).half()
        out.append((a, b))
    return out


def prepare(case, seed):
    hg.load()
    state = {"case": case, "ab": _inputs(case, seed), "stream": torch.cuda.current_stream().cuda_stream}
    if case["kind"] == "oneshot":
        return state
    prods = _products(case)
    state["c"] = [torch.empty((m, n), dtype=torch.float16, device="cuda") for m, n, _ in prods]
    layouts = [hg.Layouts.make(b_col_major=case["tn"], lda=a.shape[1]) for a, _ in state["ab"]]
    state["layouts"] = layouts
    state["pointers"] = [(a.data_ptr(), b.data_ptr(), c.data_ptr()) for (a, b), c in zip(state["ab"], state["c"])]
    if case["kind"] == "batch":
        state["plans"] = [hg.Plan(*prods[0], layouts[0])]
        state["sets"] = state["plans"][0].pointer_sets(state["pointers"])
    elif case["kind"] != "static":
        state["plans"] = [hg.Plan(*p, lay) for p, lay in zip(prods, layouts)]
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "oneshot":
        a, b = state["ab"][0]
        return hg.hgemm(a, b, b_col_major=case["tn"])
    if kind == "batch":
        state["plans"][0].run_many(case["count"], state["sets"], state["stream"])
    elif kind == "static":
        a, b, c = state["pointers"][0]
        hg.run_static(case["m"], case["n"], case["k"], state["layouts"][0], a, b, c, state["stream"])
    else:
        for plan, (a, b, c) in zip(state["plans"], state["pointers"]):
            plan.run(a, b, c, state["stream"])
    return state["c"]


def work(case):
    prods = _products(case)
    return {"bytes": sum(2.0 * (m * k + k * n + m * n) for m, n, k in prods), "flops": sum(2.0 * m * n * k for m, n, k in prods)}


def tolerance(case):
    """Products are summed in 32 bits and rounded once to 16: every case is 2.1e-4 from its value in 64 bits (measured), the
    rounding itself; two correct orders of summation differ where a sum lies close to the middle of two 16-bit values, and
    then by one unit in the last place (2^-10 of the value).  Four times each."""
    return {"rel": 8e-4, "max": 4e-3}


def exact(case, seed):
    out = []
    for (m, n, k), (a, b) in zip(_products(case), _inputs(case, seed)):
        b = b.double()
        out.append(torch.matmul(a[:, :k].double(), b.t() if case["tn"] else b))
    return out[0] if case["kind"] == "oneshot" else out
