"""The library's representative calls, for timing and for comparing two builds.

A case is a dict of plain values.  ``listed()`` names the calls that users make
most, from the smallest to the largest; ``draw(rng)`` gives further cases of
the same ranges; ``prepare(case, seed)`` makes what a program holds before the
call (inputs on the GPU, kept outputs, a batch plan); ``run(state)`` is one
pass through the public entry points and returns what it computed;
``work(case)`` is the bytes and operations that the pass cannot do without;
``exact(case, seed)`` is the pass in float64, written in plain torch.

Five kinds of pass:

* ``vec``   the paper's vector operations in a row, as an iterative solver
            issues them: copy, x = a y + b z, <y, z>, ||z||.  ``start`` > 0
            takes every vector from that element of a longer one (a slice).
* ``gemv``  one matrix-vector product, either layout, either transpose, with
            any leading dimension (``pad`` entries between the lines), alpha and
            beta, and increments of x and y.
* ``grad``  y = A x through autograd, forward and backward (dA and dx).
* ``cg``    one conjugate-gradient-style iteration on a dense symmetric matrix:
            the fused q = A p, <p, q>; the fused x, r update with <r, r>; p.
* ``batch`` one run of a plan of many uneven GEMVs and inner products.
"""
import math
import random

import torch

from paper_1409_0669_amd import autograd, batch, composite, ops

TYPES = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}
SIZE = {"f64": 8, "f32": 4, "bf16": 2}
ALPHA, BETA = 0.75, -1.25  # the factors of the vector pass's scaled addition


def listed():
    return [
        # a short vector: a small system's solver, where each call's latency is the cost
        {"name": "vec_1e3_f64", "kind": "vec", "dtype": "f64", "acc": "plain", "n": 1000, "start": 0},
        # the paper's smallest size class, an odd length, float32 summed with compensation
        {"name": "vec_1e5_f32", "kind": "vec", "dtype": "f32", "acc": "compensated", "n": 100003, "start": 0},
        # slices of packed reduced-precision buffers: they start on any element
        {"name": "vec_1e7_bf16_slice", "kind": "vec", "dtype": "bf16", "acc": "plain", "n": 10000019, "start": 3},
        # the paper-scale vectors, in the paper's precision, far outside the caches
        {"name": "vec_2p26_f64", "kind": "vec", "dtype": "f64", "acc": "plain", "n": 1 << 26, "start": 0},
        # a small dense operator applied again and again
        {"name": "gemv_small_f64", "kind": "gemv", "dtype": "f64", "acc": "plain", "m": 200, "n": 256,
         "layout": "row", "trans": False, "pad": 0, "alpha": 1.0, "beta": 0.0, "incx": 1, "incy": 1},
        # the adjoint product of a row-major matrix at the paper's 4096 x 4096
        {"name": "gemv_4096_f32_trans", "kind": "gemv", "dtype": "f32", "acc": "plain", "m": 4096, "n": 4096,
         "layout": "row", "trans": True, "pad": 0, "alpha": 1.0, "beta": 0.0, "incx": 1, "incy": 1},
        # reduced-precision storage, compensated, contiguous rows of an odd length
        {"name": "gemv_ragged_bf16", "kind": "gemv", "dtype": "bf16", "acc": "compensated", "m": 3001, "n": 4099,
         "layout": "row", "trans": False, "pad": 0, "alpha": 1.0, "beta": 0.0, "incx": 1, "incy": 1},
        # the BLAS form as other programs call it: alpha, beta, x a strided column, Fortran storage
        {"name": "gemv_blas_f64", "kind": "gemv", "dtype": "f64", "acc": "plain", "m": 1501, "n": 1200,
         "layout": "col", "trans": False, "pad": 3, "alpha": 0.5, "beta": 0.5, "incx": 3, "incy": 1},
        # the paper-scale matrix-vector product
        {"name": "gemv_16384_f64", "kind": "gemv", "dtype": "f64", "acc": "plain", "m": 16384, "n": 16384,
         "layout": "row", "trans": False, "pad": 0, "alpha": 1.0, "beta": 0.0, "incx": 1, "incy": 1},
        # a layer's forward and backward, tall float32 matrix
        {"name": "grad_16384x2048_f32", "kind": "grad", "dtype": "f32", "acc": "plain", "m": 16384, "n": 2048},
        # one iteration of the composite workload (double precision)
        {"name": "cg_8192_f64", "kind": "cg", "dtype": "f64", "acc": "plain", "n": 8192},
        # the uneven batch: sizes spread over their logarithm, reduced precision with compensation
        {"name": "batch_512_4096_bf16", "kind": "batch", "dtype": "bf16", "acc": "compensated", "gemvs": 512,
         "dots": 4096, "sizes": 0},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("vec", "vec", "gemv", "gemv", "gemv", "grad", "cg", "batch"))
    dtype = rng.choice(("f64", "f32") if kind in ("grad", "cg") else ("f64", "f32", "bf16"))
    c = {"kind": kind, "dtype": dtype, "acc": rng.choice(("plain", "compensated"))}
    if kind == "vec":
        c["n"] = _log(rng, 1000, 1 << 26)
        c["start"] = rng.choice((0, 0, 1, 2, 3, 5))
    elif kind in ("gemv", "grad"):
        c["m"], c["n"] = _log(rng, 64, 16384), _log(rng, 64, 16384)
        if kind == "gemv":
            c["layout"], c["trans"] = rng.choice(("row", "col")), rng.random() < 0.5
            c["pad"] = rng.choice((0, 0, 0, 1, 3, 8))
            blas = rng.random() < 0.3
            c["alpha"], c["beta"] = (0.5, rng.choice((0.0, 0.5))) if blas else (1.0, 0.0)
            c["incx"], c["incy"] = (rng.choice((1, 1, 3)), rng.choice((1, 1, 2))) if blas else (1, 1)
    elif kind == "cg":
        c["n"] = _log(rng, 64, 8192)
    else:
        most = {"f64": 128, "f32": 256, "bf16": 512}[dtype]
        c["gemvs"] = _log(rng, 4, most)
        c["dots"], c["sizes"] = c["gemvs"] * rng.choice((1, 4, 8)), rng.randrange(1 << 20)
    return c


def _batch_sizes(case):
    """The uneven batch's sizes: matrices of 32 to 4096 rows and columns, vectors of 10^3 to 10^6."""
    r = random.Random(case["sizes"])
    mn = [(_log(r, 32, 4096), _log(r, 32, 4096)) for _ in range(case["gemvs"])]
    return mn, [_log(r, 1000, 1000000) for _ in range(case["dots"])]


def _offsets(sizes):
    """Starts of problems packed into one buffer, each on a multiple of 64 elements, and its length."""
    at, starts = 0, []
    for s in sizes:
        starts.append(at)
        at += (s + 63) // 64 * 64
    return starts, at


def _uniform(g, n, dtype):
    """Uniform values on [-1, 1) of a storage type."""
    t = torch.rand(n, generator=g, dtype=torch.float32 if dtype != "f64" else torch.float64, device="cuda")
    return t.mul_(2.0).sub_(1.0).to(TYPES[dtype])


def _lines(case):
    """(lines, entries of a line, leading dimension) of a GEMV case's matrix."""
    lines, k = (case["m"], case["n"]) if case["layout"] == "row" else (case["n"], case["m"])
    return lines, k, k + case["pad"]


def _inputs(case, seed):
    """The case's inputs, from the seed alone."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    kind, dt = case["kind"], case["dtype"]
    s = {"case": case, "kind": kind, "acc": case["acc"]}
    if kind == "vec":
        n, at = case["n"], case["start"]
        y = _uniform(g, n + at, dt)
        # two vectors of one problem (a direction and its image): correlated
        z = _uniform(g, n + at, dt).mul_(0.5).add_(y, alpha=0.5)
        s["y"], s["z"] = y[at:], z[at:]
        s["x"], s["copy"] = torch.empty_like(y)[at:], torch.empty_like(y)[at:]
    elif kind == "gemv":
        m, n = case["m"], case["n"]
        lines, k, ld = _lines(case)
        a = _uniform(g, lines * ld, dt).view(lines, ld)[:, :k]
        s["A"] = a if case["layout"] == "row" else a.t()
        rows, cols = (n, m) if case["trans"] else (m, n)
        s["x"] = _uniform(g, cols * case["incx"], dt)[::case["incx"]]
        out = "f64" if dt == "f64" else "f32"
        # a call with beta reads y, one with an increment writes into a kept vector
        kept = case["beta"] != 0.0 or case["incy"] != 1
        s["y"] = _uniform(g, rows * case["incy"], out)[::case["incy"]] if kept else None
    elif kind == "grad":
        m, n = case["m"], case["n"]
        s["A"] = _uniform(g, m * n, dt).view(m, n).requires_grad_()
        s["x"] = _uniform(g, n, dt).requires_grad_()
        s["ybar"] = _uniform(g, m, dt)
    elif kind == "cg":
        n = case["n"]
        a = torch.randn(n, n, generator=g, dtype=torch.float64, device="cuda")
        a = (a + a.t()).mul_(0.05 / math.sqrt(2.0 * n))  # symmetric, eigenvalues near 1: passes stay bounded
        a.diagonal().add_(1.0)
        s["A"] = a.to(TYPES[dt])
        for v in ("x", "p", "r"):
            s[v] = _uniform(g, n, dt)
        s["q"] = torch.empty_like(s["x"])
    else:
        mn, d = _batch_sizes(case)
        a_at, a_n = _offsets([m * n for m, n in mn])
        x_at, x_n = _offsets([n for _, n in mn])
        d_at, d_n = _offsets(d)
        a, x, u = _uniform(g, a_n, dt), _uniform(g, x_n, dt), _uniform(g, d_n, dt)
        w = _uniform(g, d_n, dt).mul_(0.5).add_(u, alpha=0.5)
        s["gemvs"] = [(a[i:i + m * n].view(m, n), x[j:j + n]) for (m, n), i, j in zip(mn, a_at, x_at)]
        s["dots"] = [(u[i:i + n], w[i:i + n]) for n, i in zip(d, d_at)]
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    if s["kind"] == "batch":
        out = torch.float64 if case["dtype"] == "f64" else torch.float32
        s["ys"] = torch.empty(sum(a.shape[0] for a, _ in s["gemvs"]), dtype=out, device="cuda")
        s["outs"] = torch.empty(len(s["dots"]), dtype=out, device="cuda")
        gemvs, at = [], 0
        for a, x in s["gemvs"]:
            gemvs.append((a, x, s["ys"][at:at + a.shape[0]]))
            at += a.shape[0]
        dots = [(u, w, s["outs"][i:i + 1]) for i, (u, w) in enumerate(s["dots"])]
        s["plan"] = batch.BatchPlan(gemvs, dots, acc=case["acc"])
    return s


def run(s):
    kind, acc = s["kind"], s["acc"]
    if kind == "vec":
        ops.copy(s["y"], out=s["copy"])
        ops.axpby(ALPHA, s["y"], BETA, s["z"], out=s["x"])
        return {"copy": s["copy"], "x": s["x"], "dot": ops.dot(s["y"], s["z"], acc=acc),
                "nrm2": ops.nrm2(s["z"], acc=acc)}
    if kind == "gemv":
        c = s["case"]
        return ops.gemv(s["A"], s["x"], trans=c["trans"], acc=acc, out=s["y"], alpha=c["alpha"], beta=c["beta"])
    if kind == "grad":
        y = autograd.gemv(s["A"], s["x"], acc)
        dA, dx = torch.autograd.grad(y, (s["A"], s["x"]), s["ybar"])
        return {"y": y, "dA": dA, "dx": dx}
    if kind == "cg":
        q, pq = composite.gemv_dot_fused(s["A"], s["p"], acc=acc, q=s["q"])
        rr = composite.cg_step_fused(1.0, s["x"], s["p"], s["r"], q, acc=acc)
        ops.axpby(1.0, s["r"], 1.0, s["p"], out=s["p"])
        return {"q": q, "pq": pq, "x": s["x"], "r": s["r"], "rr": rr, "p": s["p"]}
    s["plan"].run()
    return {"y": s["ys"], "dots": s["outs"]}


def work(case):
    """Each call's inputs read once and its outputs written once; a multiply and an add per product."""
    kind, e = case["kind"], SIZE[case["dtype"]]
    o = max(e, 4)  # a reduction's output entry
    if kind == "vec":
        n = case["n"]
        return {"bytes": 8 * n * e + 2 * o, "flops": 7 * n}
    if kind in ("gemv", "grad"):
        m, n = case["m"], case["n"]
        if kind == "grad":  # A read by each product, dA written
            return {"bytes": 3 * m * n * e + (3 * m + 3 * n) * e, "flops": 5 * m * n}
        rows, cols = (n, m) if case["trans"] else (m, n)
        return {"bytes": m * n * e + cols * e + rows * o * (1 if case["beta"] == 0.0 else 2), "flops": 2 * m * n}
    if kind == "cg":
        n = case["n"]
        return {"bytes": n * n * e + 11 * n * e, "flops": 2 * n * n + 11 * n}
    mn, d = _batch_sizes(case)
    return {"bytes": sum(m * n * e + n * e + m * o for m, n in mn) + sum(2 * n * e + o for n in d),
            "flops": sum(2 * m * n for m, n in mn) + sum(2 * n for n in d)}


def exact(case, seed):
    s = _inputs(case, seed)
    kind = s["kind"]
    if kind == "vec":
        y, z = s["y"].double(), s["z"].double()
        return {"copy": y, "x": ALPHA * y + BETA * z, "dot": torch.dot(y, z), "nrm2": torch.linalg.vector_norm(z)}
    if kind == "gemv":
        a = s["A"].double()
        y = case["alpha"] * torch.mv(a.t() if case["trans"] else a, s["x"].double())
        return y + case["beta"] * s["y"].double() if case["beta"] != 0.0 else y
    if kind == "grad":
        a, x, ybar = s["A"].detach().double(), s["x"].detach().double(), s["ybar"].double()
        return {"y": torch.mv(a, x), "dA": torch.outer(ybar, x), "dx": torch.mv(a.t(), ybar)}
    if kind == "cg":
        a, x, p, r = (s[k].double() for k in ("A", "x", "p", "r"))
        q = torch.mv(a, p)
        x, r = x + p, r - q
        return {"q": q, "pq": torch.dot(p, q), "x": x, "r": r, "rr": torch.dot(r, r), "p": r + p}
    ys = [torch.mv(a.double(), x.double()) for a, x in s["gemvs"]]
    dots = [torch.dot(u.double(), w.double()) for u, w in s["dots"]]
    return {"y": torch.cat(ys), "dots": torch.stack(dots)}
