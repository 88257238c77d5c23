"""Timed workloads of the merge-path SpMV library, each through the public Python binding.

A case is a dict of plain values:

    kind    "spmv"      one y = A x on a kept plan
            "spmm"      one Y = A X over k right-hand sides
            "pagerank"  `iters` power iterations on a kept plan
            "ppr"       personalised PageRank of k sources, `iters` iterations
            "multi"     PageRank of many graphs on one diagonal
            "grad"      differentiable PageRank: forward, loss, backward
            "bicgstab"  (I - alpha P) x = (1 - alpha)/n solved to 1e-12
            "plan"      what a new matrix costs: plan, transpose, first SpMV
    graph   "rmat" (2^scale vertices, 16 edge draws each) or "cl" (Chung-Lu,
            any n, `deg` edge draws per vertex, 10 % empty rows)
    dtype   "f32" or "f64"
    stripes, desc_bits, sigma, lanes   plan options (0 = the library's default)

Inputs are drawn on the GPU from the seed alone; the graphs follow the
recipes of graphgen (R-MAT a, b, c = 0.57, 0.19, 0.19; Chung-Lu with source
exponent 2.1), duplicates merged and thinned to a number of edges that depends
on the case alone, rows = destinations, values 1/outdeg.
"""
import math

import torch

import paper_2605_07391_amd.merbit as mb
from paper_2605_07391_amd.autograd import DiffPageRank

ALPHA = 0.85
DTYPES = {"f32": torch.float32, "f64": torch.float64}


def _case(name, kind, dtype, graph, **kw):
    c = {"name": name, "kind": kind, "dtype": dtype, "graph": graph, "scale": 0, "n": 0, "deg": 0,
         "graphs": 0, "k": 0, "iters": 0, "stripes": 0, "desc_bits": 32, "sigma": 0, "lanes": 0}
    c.update(kw)
    return c


def listed():
    return [
        # a small web graph or road-map tile: one product, bound by launches
        _case("spmv_cl10k_f32", "spmv", "f32", "cl", n=10_000, deg=10),
        # the solver's product: FP64, a ragged size, library defaults
        _case("spmv_cl700k_f64", "spmv", "f64", "cl", n=700_001, deg=12),
        # the largest graph of the benchmark with the library's default plan
        _case("spmv_rmat22_f32", "spmv", "f32", "rmat", scale=22),
        # ranks of a small graph, as a service computes them on request
        _case("pagerank_cl10k_f32", "pagerank", "f32", "cl", n=10_000, deg=10, iters=20),
        # the benchmark's headline: PageRank on the configuration it tunes to
        _case("pagerank_rmat22_f32_s8", "pagerank", "f32", "rmat", scale=22, iters=20, stripes=8,
              desc_bits=64, sigma=28, lanes=512),
        # a block of a few vectors (block solvers, feature propagation), FP64
        _case("spmm_cl100k_f64_k5", "spmm", "f64", "cl", n=100_003, deg=8, k=5),
        # feature propagation over a full-width block
        _case("spmm_rmat20_f32_k64", "spmm", "f32", "rmat", scale=20, k=64),
        # recommendations for a batch of users
        _case("ppr_rmat18_f32_k16", "ppr", "f32", "rmat", scale=18, k=16, iters=10),
        # a batch of unrelated graphs ranked at once
        _case("multi64_f32_s8", "multi", "f32", "cl", graphs=64, deg=8, iters=10, stripes=8,
              desc_bits=64, sigma=24, lanes=512),
        # one training step of learned edge weights: forward and backward
        _case("grad_rmat20_f32", "grad", "f32", "rmat", scale=20, iters=20),
        # PageRank as a linear system, solved to convergence in FP64
        _case("bicgstab_rmat20_f64", "bicgstab", "f64", "rmat", scale=20),
        # a new matrix: everything a user pays before and with the first product
        _case("plan_rmat20_f32", "plan", "f32", "rmat", scale=20),
    ]


def draw(rng):
    kind = rng.choice(["spmv", "spmv", "spmm", "spmm", "pagerank", "ppr", "multi", "grad",
                       "bicgstab", "plan"])
    dtype = rng.choice(["f32", "f64"])
    kw = {}
    if kind == "bicgstab":
        dtype = "f64"  # the solver's runs are FP64 (its tolerance is below FP32)
    top = 2_000_000 if kind in ("spmv", "pagerank", "plan") else 700_000
    if kind == "multi":
        graph = "cl"
        kw.update(graphs=rng.randint(3, 64), deg=8)
    elif rng.random() < 0.4:
        graph = "rmat"
        kw["scale"] = rng.randint(10, int(math.log2(top)))
    else:
        graph = "cl"
        kw.update(n=int(math.exp(rng.uniform(math.log(1000), math.log(top)))), deg=rng.randint(4, 16))
    if kind in ("spmm", "ppr"):
        kw["k"] = int(math.exp(rng.uniform(0.0, math.log(64.999))))
    if kind in ("pagerank", "ppr", "multi", "grad"):
        kw["iters"] = rng.randint(5, 25)
    if kind in ("spmv", "pagerank", "multi") and rng.random() < 0.4:
        kw["stripes"] = rng.choice([4, 8])
        if rng.random() < 0.5:
            kw.update(desc_bits=64, lanes=512, sigma=rng.choice([16, 24] if dtype == "f32" else [14, 20]))
    elif kind == "grad" and rng.random() < 0.3:
        kw["stripes"] = 8
    c = _case("", kind, dtype, graph, **kw)
    del c["name"]
    return c


# ----------------------------------------------------------------- inputs --

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1_000_003 + 17)
    return g


def _rmat_keys(scale, m, gen):
    n = 1 << scale
    row = torch.zeros(m, dtype=torch.int32, device="cuda")
    col = torch.zeros(m, dtype=torch.int32, device="cuda")
    for _ in range(scale):
        u = torch.rand(m, generator=gen, device="cuda")
        row.mul_(2).add_(u >= 0.76)
        col.mul_(2).add_(((u >= 0.57) & (u < 0.76)) | (u >= 0.95))
    return row.long() * n + col.long()


def _cl_keys(sizes, deg, empty, gen):
    """Chung-Lu graphs of the given sizes on one diagonal: source weights
    (i + 1)^(-1/1.1) by inverse distribution, targets uniform over the
    vertices that may have in-edges."""
    sz = torch.tensor(sizes, dtype=torch.int64, device="cuda")
    off = torch.cumsum(sz, 0) - sz
    n, m = int(sum(sizes)), deg * int(sum(sizes))
    g = torch.repeat_interleave(torch.arange(len(sizes), device="cuda"), sz * deg, output_size=m)
    s = sz[g].double()
    e = 1.0 - 1.0 / 1.1
    u = torch.rand(m, generator=gen, device="cuda", dtype=torch.float64)
    src = ((u * ((s + 1.0) ** e - 1.0) + 1.0) ** (1.0 / e)).long() - 1
    src = torch.minimum(src.clamp_(min=0), sz[g] - 1) + off[g]
    dst = (torch.rand(m, generator=gen, device="cuda", dtype=torch.float64) * s).long()
    dst = torch.minimum(dst, sz[g] - 1) + off[g]
    return (dst * n + src)[~empty[dst]]


def _sizes(case):
    if not case["graphs"]:
        return [case["n"]]
    # vertex counts log-uniform in [1,000, 200,000], the same for every seed
    # (a service's batch changes its edges and values, its shape class stays)
    g = torch.Generator().manual_seed(40 + case["graphs"])
    u = torch.rand(case["graphs"], generator=g, dtype=torch.float64)
    return [int(math.exp(math.log(1000) + float(v) * math.log(200.0))) for v in u]


def _shape(case):
    """Vertices and edges: as many edges for every seed, a little under what
    the draws give once their duplicates are merged."""
    if case["graph"] == "rmat":
        return 1 << case["scale"], 15 << case["scale"]
    n = sum(_sizes(case))
    return n, int((0.8 if case["graphs"] else 0.85) * case["deg"] * n)


class _Matrix:
    """CSR pattern (row_ptr, col int32), the row of each nonzero, values."""

    def __init__(self, case, seed, gen):
        dt = DTYPES[case["dtype"]]
        self.sizes = _sizes(case)
        n, edges = _shape(case)
        empty = torch.rand(n, generator=gen, device="cuda") < 0.1
        key = torch.empty(0, dtype=torch.int64, device="cuda")
        while key.numel() < edges:  # duplicates are merged: small graphs need further draws
            more = (_rmat_keys(case["scale"], 16 * n, gen) if case["graph"] == "rmat"
                    else _cl_keys(self.sizes, case["deg"], empty, gen))
            key = torch.unique(torch.cat([key, more]))
        keep = torch.randperm(key.numel(), generator=gen, device="cuda")[:edges]
        key = key[torch.sort(keep).values]
        if case["kind"] == "bicgstab":  # I - alpha P: the diagonal is stored
            diag = torch.arange(n, device="cuda") * (n + 1)
            col = key % n
            on = torch.bincount(col, minlength=n).double()
            full = torch.unique(torch.cat([key, diag]))
            at = torch.searchsorted(full, key)
            val = torch.zeros(full.numel(), dtype=torch.float64, device="cuda")
            val[at] = -ALPHA / on[col]
            val[torch.searchsorted(full, diag)] += 1.0
            key = full
        row, col = key // n, key % n
        if case["kind"] != "bicgstab":
            val = 1.0 / torch.bincount(col, minlength=n).double()[col]
        self.n, self.m = n, key.numel()
        self.row, self.col = row.int(), col.int()
        self.row_ptr = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
        self.row_ptr[1:] = torch.cumsum(torch.bincount(row, minlength=n), 0).int()
        self.val = val.to(dt)


def _inputs(case, seed):
    """The matrix and the vectors of one case, from the seed alone."""
    gen = _gen(seed)
    A = _Matrix(case, seed, gen)
    dt, n, kind = DTYPES[case["dtype"]], A.n, case["kind"]

    def uniform(*shape):
        return torch.rand(*shape, generator=gen, device="cuda", dtype=dt) * 2 - 1

    s = {"A": A}
    if kind in ("spmv", "plan"):
        s["x"] = uniform(n)
    elif kind == "spmm":
        s["x"] = uniform(n, case["k"])
    elif kind == "pagerank":
        s["x0"] = torch.full((n,), 1.0 / n, dtype=dt, device="cuda")
    elif kind == "ppr":
        s["sources"] = torch.randperm(n, generator=gen, device="cuda")[:case["k"]].cpu().numpy()
    elif kind == "multi":
        sz = torch.tensor(A.sizes, dtype=torch.int64)
        s["graph_ptr"] = torch.cat([torch.zeros(1, dtype=torch.int64), torch.cumsum(sz, 0)]).numpy()
        szd = sz.cuda()
        s["x0"] = torch.repeat_interleave(1.0 / szd.double(), szd).to(dt)
    elif kind == "grad":
        s["w"] = (1.5 - torch.rand(A.m, generator=gen, device="cuda", dtype=dt))  # (0.5, 1.5]
        t = torch.rand(n, generator=gen, device="cuda", dtype=dt)
        s["t"] = t / t.sum()
    elif kind == "bicgstab":
        s["b"] = torch.full((n,), (1.0 - ALPHA) / n, dtype=dt, device="cuda") * (uniform(n) * 0.5 + 1)
    return s


def _plan(A, case):
    return mb.Plan(A.row_ptr, A.col, A.val, A.n, sigma=case["sigma"], block_lanes=case["lanes"],
                   stripes=case["stripes"], desc_bits=case["desc_bits"])


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"], A, kind = dict(case), s["A"], case["kind"]
    A.row = None  # only exact() reads it
    if kind == "grad":
        s["op"] = DiffPageRank(A.row_ptr, A.col, A.n, dtype=DTYPES[case["dtype"]], alpha=ALPHA,
                               max_iter=case["iters"], stripes=case["stripes"])
        s["w"].requires_grad_(True)
    elif kind != "plan":
        s["plan"] = _plan(A, case)
    if kind in ("spmv", "spmm"):
        s["y"] = torch.empty_like(s["x"])  # a loop writes its products into one buffer
    elif kind in ("pagerank", "multi"):
        s["x"] = torch.empty_like(s["x0"])
    elif kind == "bicgstab":
        s["x"] = torch.empty_like(s["b"])
    return s


def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind == "spmv":
        return s["plan"].spmv(s["x"], out=s["y"])
    if kind == "spmm":
        return s["plan"].spmm(s["x"], out=s["y"])
    if kind == "pagerank":
        s["x"].copy_(s["x0"])
        it, _, _ = s["plan"].pagerank(s["x"], ALPHA, max_iter=case["iters"])
        return {"x": s["x"], "iters": it}
    if kind == "ppr":
        X, it, _, _ = s["plan"].pagerank_personalized(s["sources"], alpha=ALPHA,
                                                      max_iter=case["iters"])
        return {"x": X, "iters": it}
    if kind == "multi":
        s["x"].copy_(s["x0"])
        it, _, _ = s["plan"].pagerank_multi(s["graph_ptr"], s["x"], ALPHA, max_iter=case["iters"])
        return {"x": s["x"], "iters": it}
    if kind == "grad":
        s["w"].grad = None
        x = s["op"](s["w"])
        loss = 0.5 * ((x - s["t"]) ** 2).sum()
        loss.backward()
        return {"x": x.detach(), "grad": s["w"].grad}
    if kind == "bicgstab":
        s["x"].zero_()
        it, _, status = s["plan"].bicgstab(s["b"], s["x"], tol=1e-12, max_iter=200)
        return {"x": s["x"], "iters": it, "converged": status == "converged"}
    A = s["A"]
    plan = _plan(A, case)
    row_t, col_t, perm = plan.transpose()
    y = plan.spmv(s["x"])
    plan.close()
    return {"y": y, "row_t": row_t, "col_t": col_t, "perm": perm}


# ------------------------------------------------------ 64-bit reference --

def _sums(values, ptr):
    """Sum of each segment values[ptr[i] : ptr[i + 1]] along the first axis."""
    return torch.segment_reduce(values, "sum", offsets=ptr.long(), axis=0, unsafe=True)


class _Product:
    """x -> A x in float64 (x may have columns), A in CSR order of its rows."""

    def __init__(self, ptr, col, val):
        self.ptr, self.col, self.val = ptr, col, val

    def __call__(self, x):
        if x.dim() == 1:
            return _sums(self.val * x[self.col], self.ptr)
        return torch.cat([_sums(self.val[:, None] * x[:, j:j + 8][self.col], self.ptr)
                          for j in range(0, x.shape[1], 8)], 1)


def exact(case, seed):
    s = _inputs(case, seed)
    A, kind, iters = s["A"], case["kind"], case["iters"]
    val, n = A.val.double(), A.n
    dangling = (torch.bincount(A.col, minlength=n) == 0).double()
    product = _Product(A.row_ptr, A.col, val)
    if kind in ("spmv", "spmm"):
        return product(s["x"].double())
    if kind == "pagerank":
        x = s["x0"].double()
        for _ in range(iters):
            x = ALPHA * product(x) + (ALPHA * (dangling * x).sum() + 1 - ALPHA) / n
        return {"x": x, "iters": None}
    if kind == "ppr":
        src = torch.as_tensor(s["sources"], device="cuda")
        at = (src, torch.arange(case["k"], device="cuda"))
        x = torch.zeros(n, case["k"], dtype=torch.float64, device="cuda")
        x[at] = 1.0
        for _ in range(iters):
            d = (dangling[:, None] * x).sum(0)
            x = ALPHA * product(x)
            x[at] += ALPHA * d + 1 - ALPHA
        return {"x": x, "iters": None}
    if kind == "multi":
        sz = torch.tensor(A.sizes, dtype=torch.int64, device="cuda")
        g = torch.repeat_interleave(torch.arange(len(A.sizes), device="cuda"), sz)
        x = s["x0"].double()
        for _ in range(iters):
            d = torch.zeros(len(A.sizes), dtype=torch.float64, device="cuda")
            d.index_add_(0, g, dangling * x)
            x = ALPHA * product(x) + ((ALPHA * d + 1 - ALPHA) / sz)[g]
        return {"x": x, "iters": None}
    if kind == "grad":
        w, t = s["w"].double(), s["t"].double()
        col, row = A.col.long(), A.row.long()

        order = torch.argsort(col, stable=True)  # the nonzeros by column
        ptr_t = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
        ptr_t[1:] = torch.cumsum(torch.bincount(col, minlength=n), 0)
        cs = _sums(w[order], ptr_t)
        P = w / cs[col]
        product, product_t = _Product(A.row_ptr, A.col, P), _Product(ptr_t, row[order], P[order])
        x = torch.full((n,), 1.0 / n, dtype=torch.float64, device="cuda")
        for _ in range(iters):
            x = ALPHA * product(x) + (ALPHA * (dangling * x).sum() + 1 - ALPHA) / n
        g = x - t
        lam = g.clone()
        for _ in range(iters):
            lam = g + ALPHA * product_t(lam) + ALPHA / n * lam.sum() * dangling
        G = ALPHA * lam[row] * x[col]
        return {"x": x, "grad": (G - _sums((G * P)[order], ptr_t)[col]) / cs[col]}
    if kind == "bicgstab":
        # x = b + (I - A) x, a contraction of factor alpha in the 1-norm
        b = s["b"].double()
        x = b.clone()
        for _ in range(260):
            x = x + (b - product(x))
        return {"x": x, "iters": None, "converged": None}
    return {"y": product(s["x"].double()), "row_t": None, "col_t": None, "perm": None}


# ------------------------------------------------------- compulsory work --

def work(case):
    """Bytes and operations a pass cannot do without: the matrix (values,
    column indices, row lengths) and each vector read or written once per
    product."""
    vs = 4 if case["dtype"] == "f32" else 8
    n, m = _shape(case)
    if case["kind"] == "bicgstab":
        m += n  # the diagonal
    matrix, kind = m * (vs + 4) + 4 * n, case["kind"]
    k = max(1, case["k"])
    step = {"bytes": matrix + 2 * n * k * vs, "flops": 2 * m * k}
    if kind in ("spmv", "spmm"):
        return step
    if kind in ("pagerank", "ppr", "multi"):
        return {q: v * case["iters"] for q, v in step.items()}
    if kind == "grad":
        # both fixed points; the weights' normalisation, the transposed
        # values and the two value gradients, each over the nonzeros once
        extra = m * (4 * vs + 8)
        return {"bytes": 2 * case["iters"] * step["bytes"] + extra,
                "flops": 2 * case["iters"] * step["flops"] + 8 * m}
    if kind == "bicgstab":
        # ten iterations at least (the first convergence test): two products
        # and about twenty vector passes each
        return {"bytes": 10 * (2 * step["bytes"] + 20 * n * vs), "flops": 10 * (2 * step["flops"] + 20 * n)}
    # plan: the CSR once, the transpose's arrays written, one product
    return {"bytes": step["bytes"] + m * 8 + 4 * n, "flops": step["flops"]}
