"""Workloads of the library's public entry points, for timing and comparison.

A case is a dict of plain values; its "path" names the call it stands for:

    spmv      y = A x with a kept handle, vectors in the caller's ids
    build     format build, one product, release: a matrix used once
    pagerank  PageRank to a tolerance on a kept handle
    job       build, a fixed number of PageRank iterations, release (bench.py's step)
    hits      HITS iterations on the 2n x 2n block matrix
    rwr       random walk with restart, k queries at once, to a tolerance
    spmm      Y = A X with a kept handle, k right-hand sides in the caller's ids
    multi     RWR on many graphs per launch, one query each
    diff      learned edge weights: scores, loss and the gradient of theta

Graphs are seeded and made on the GPU: R-MAT (a .57, b .19, c .19; for n that is
no power of two the ids of the next larger power of two are scaled down), Chung-Lu
(exponent 2.1, in-weights an independent permutation of the out-weights, ids
permuted) and uniform.  "draws" is the number of edges drawn; repeated ones are
dropped, so a matrix holds somewhat fewer entries.
"""
import math

import numpy as np
import torch

from paper_1103_2405_amd import DeviceCsr, TiledMatrix, rwr_multi
from paper_1103_2405_amd.rwr_grad import EdgeWeightedRWR

DAMP = 0.85
C64 = float(np.float32(DAMP))  # the entry points take c as a 32-bit float
FORMATS = {"tiles": {}, "panels": {"panels": -1}, "coo": {"kernel": "coo"}}


def listed():
    return [
        # a product on a small graph (scale-14 R-MAT of the benchmark): launches and latency
        {"name": "spmv-rmat14", "path": "spmv", "graph": "rmat", "n": 1 << 14, "draws": 1 << 18, "format": "tiles"},
        # the benchmark's matrix, row panels: the largest product
        {"name": "spmv-cl23-panels", "path": "spmv", "graph": "chung-lu", "n": 1 << 23, "draws": 1 << 27,
         "format": "panels"},
        # the coordinate kernel on the benchmark's matrix without a power law: 16 entries a row
        {"name": "spmv-coo-uniform20", "path": "spmv", "graph": "uniform", "n": 1 << 20, "draws": 1 << 24,
         "format": "coo"},
        # a matrix that is built, used and dropped: default format, scale-20 R-MAT of the benchmark
        {"name": "build-rmat20", "path": "build", "graph": "rmat", "n": 1 << 20, "draws": 1 << 24,
         "format": "tiles"},
        # PageRank of a small graph to a tolerance, its residual read every 5 iterations
        {"name": "pagerank-rmat14", "path": "pagerank", "graph": "rmat", "n": 1 << 14, "draws": 1 << 18,
         "format": "tiles", "tol": 1e-6, "check": 5},
        # the benchmark's whole step
        {"name": "job-cl23", "path": "job", "graph": "chung-lu", "n": 1 << 23, "draws": 1 << 27, "format": "panels",
         "iters": 100},
        # HITS on the scale-20 R-MAT (2^21 rows, 32M entries)
        {"name": "hits-rmat20", "path": "hits", "graph": "rmat", "n": 1 << 20, "draws": 1 << 24, "format": "tiles",
         "iters": 15},
        # one query of a recommender: single-vector RWR on the symmetrised scale-20 R-MAT
        {"name": "rwr1-rmat20", "path": "rwr", "graph": "rmat", "n": 1 << 20, "draws": 1 << 24, "format": "tiles",
         "k": 1, "tol": 1e-6, "check": 10},
        # 32 queries in a batch on the same graph
        {"name": "rwr32-rmat20", "path": "rwr", "graph": "rmat", "n": 1 << 20, "draws": 1 << 24, "format": "tiles",
         "k": 32, "tol": 1e-6, "check": 10},
        # a rectangular matrix of odd sizes and an odd number of right-hand sides
        {"name": "spmm13-rect", "path": "spmm", "graph": "uniform", "n": 300007, "cols": 100003, "draws": 4800112,
         "format": "tiles", "k": 13},
        # the benchmark's 32 graphs of scale 10-16, edge factor 8-32, one query each
        {"name": "multi-32", "path": "multi", "graphs": 32, "lo": 10, "hi": 16, "iters": 30},
        # one training step of learned edge weights, scale-18 R-MAT, 4 features an edge
        {"name": "diff-rmat18", "path": "diff", "graph": "rmat", "n": 1 << 18, "draws": 1 << 22, "features": 4,
         "iters": 30, "every": 6, "targets": 16},
    ]


def draw(rng):
    def size(lo, hi):  # log-uniform, odd
        return int(2 ** rng.uniform(lo, hi)) | 1

    path = rng.choice(["spmv", "spmv", "build", "pagerank", "job", "hits", "rwr", "rwr", "spmm", "multi", "diff"])
    graph = rng.choice(["rmat", "rmat", "chung-lu"])
    ef = rng.uniform(4, 24)
    if path == "spmv":
        fmt = rng.choice(["tiles", "panels", "coo"])
        n = size(10, 22 if fmt == "panels" else 20.5)
        return {"path": path, "graph": rng.choice(["rmat", "chung-lu", "uniform"]), "n": n, "draws": int(ef * n),
                "format": fmt}
    if path == "build":
        n = size(10, 21)
        return {"path": path, "graph": graph, "n": n, "draws": int(ef * n), "format": rng.choice(["tiles", "panels"])}
    if path == "pagerank":
        n = size(10, 21)
        return {"path": path, "graph": graph, "n": n, "draws": int(ef * n), "format": rng.choice(["tiles", "panels"]),
                "tol": 1e-6, "check": rng.choice([1, 5, 10])}
    if path == "job":
        n = size(16, 22)
        return {"path": path, "graph": graph, "n": n, "draws": int(ef * n), "format": "panels",
                "iters": rng.randint(20, 100)}
    if path == "hits":
        n = size(10, 20.5)
        return {"path": path, "graph": graph, "n": n, "draws": int(ef * n), "format": "tiles",
                "iters": rng.randint(5, 30)}
    if path == "rwr":
        n = size(10, 20)
        return {"path": path, "graph": graph, "n": n, "draws": int(min(ef, 16) * n), "format": "tiles",
                "k": rng.choice([1, 2, 7, 8, 16, 32, 37, 64]), "tol": 1e-6, "check": rng.choice([5, 10])}
    if path == "spmm":
        n = size(10, 19)
        return {"path": path, "graph": rng.choice(["rmat", "uniform"]), "n": n, "cols": size(10, 19),
                "draws": int(ef * n), "format": "tiles", "k": rng.choice([3, 8, 13, 32, 64, 70, 100])}
    if path == "multi":
        lo = rng.randint(9, 13)
        return {"path": path, "graphs": rng.randint(3, 40), "lo": lo, "hi": rng.randint(lo, 16),
                "iters": rng.randint(10, 40)}
    n = size(10, 19)
    return {"path": path, "graph": graph, "n": n, "draws": int(min(ef, 16) * n), "features": rng.randint(1, 8),
            "iters": rng.randint(5, 30), "every": rng.randint(1, 8), "targets": 16}


# ---- inputs

def _gen(seed, k=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + k)
    return g


def _rmat_ids(n, m, g):
    scale = max(1, math.ceil(math.log2(n)))
    src = torch.zeros(m, dtype=torch.int64, device="cuda")
    dst = torch.zeros_like(src)
    for _ in range(scale):
        u = torch.rand(m, device="cuda", generator=g)
        down = u >= 0.76
        right = ((u >= 0.57) & ~down) | (u >= 0.95)
        src.mul_(2).add_(down)
        dst.mul_(2).add_(right)
    if n != 1 << scale:
        src, dst = (src * n) >> scale, (dst * n) >> scale
    return src, dst


def _chung_lu_ids(n, m, g):
    w = torch.arange(1, n + 1, dtype=torch.float64, device="cuda") ** (-1.0 / 1.1)
    cap = max(1.0, n / 8)  # the benchmark's 2^20 at 2^23 nodes
    w *= m / float(w.sum())
    for _ in range(8):  # the weight above the cap goes to the others
        low = w < cap
        over = float((w.clamp(max=cap)).sum())
        if not bool(low.any()) or abs(over - m) < 0.5:
            break
        w = torch.where(low, w * ((m - cap * float((~low).sum())) / float(w[low].sum())), torch.full_like(w, cap))
    cdf = torch.cumsum((w.clamp(max=cap) * 2.0 ** 20).long(), 0)  # whole numbers: the same sums every time
    perm = [torch.randperm(n, device="cuda", generator=g) for _ in range(2)]

    def side(p):
        return p[torch.searchsorted(cdf, torch.randint(int(cdf[-1]), (m,), device="cuda", generator=g), right=True)]

    return side(perm[0]), side(perm[1])


def _edges(graph, n, cols, m, g):
    """Distinct (row, col) pairs, sorted: a graph's edges (src, dst), or a rectangular matrix' entries."""
    if graph == "uniform" or cols != n:
        src = torch.randint(0, n, (m,), device="cuda", generator=g)
        if graph == "rmat":  # skewed columns
            dst = (torch.rand(m, device="cuda", generator=g, dtype=torch.float64) ** 4 * cols).long().clamp_(max=cols - 1)
        else:
            dst = torch.randint(0, cols, (m,), device="cuda", generator=g)
    else:
        src, dst = _rmat_ids(n, m, g) if graph == "rmat" else _chung_lu_ids(n, m, g)
    return _distinct(src, dst, cols)


def _distinct(row, col, cols):
    key = torch.sort(row * cols + col)[0]
    keep = torch.ones_like(key, dtype=torch.bool)
    keep[1:] = key[1:] != key[:-1]
    key = key[keep]
    return key // cols, key % cols


def _csr(rows, cols, r, c, val):
    rp = torch.zeros(rows + 1, dtype=torch.int64, device="cuda")
    rp[1:] = torch.cumsum(torch.bincount(r, minlength=rows), 0)
    return rows, cols, rp, c.to(torch.int32), val


def _square(case, seed):
    """The path's matrix, as (rows, cols, row_ptr, col, val), and its entries' rows."""
    n, g = case["n"], _gen(seed)
    src, dst = _edges(case["graph"], n, n, case["draws"], g)
    if case["path"] == "hits":  # [[0, A^T], [A, 0]] of ones
        r, c = _distinct(torch.cat([dst, src + n]), torch.cat([src + n, dst]), 2 * n)
        return _csr(2 * n, 2 * n, r, c, torch.ones(r.numel(), device="cuda")), r
    if case["path"] in ("rwr", "diff", "multi"):  # both directions, columns scaled to sum 1
        r, c = _distinct(torch.cat([src, dst]), torch.cat([dst, src]), n)
    elif case["graph"] == "uniform":
        return _csr(n, n, src, dst, torch.rand(src.numel(), device="cuda", generator=g)), src
    else:  # PageRank: M[v][u] = 1 / outdeg(u)
        r, c = _distinct(dst, src, n)
    deg = torch.bincount(c, minlength=n).clamp(min=1)
    return _csr(n, n, r, c, (1.0 / deg.to(torch.float64)).to(torch.float32)[c]), r


def _linked(csr, least):
    """Nodes of a symmetrised graph with at least `least` entries (or, in a sparse one, the most linked)."""
    deg = csr[2][1:] - csr[2][:-1]
    at = torch.nonzero(deg >= least).flatten()
    return at if at.numel() >= 64 else torch.topk(deg, min(64, deg.numel()))[1]


def _pick(nodes, k, g):
    return nodes[torch.randperm(nodes.numel(), device="cuda", generator=g)[:k]]


def _graphs(case, seed):
    rng = np.random.RandomState(4000 + case["graphs"])  # the sizes are the case's, the graphs the seed's
    for q in range(case["graphs"]):
        n = 1 << int(rng.randint(case["lo"], case["hi"] + 1))
        one = {"path": "multi", "graph": "rmat", "n": n, "draws": n * int(rng.randint(8, 33))}
        csr, r = _square(one, int(seed) * 64 + q)
        yield csr, r, int(_pick(_linked(csr, 1), 1, _gen(seed, q))[0])


def _inputs(case, seed):
    g = _gen(seed, 7)
    d = {}
    if case["path"] == "spmm":
        r, c = _edges(case["graph"], case["n"], case["cols"], case["draws"], g)
        d["csr"], d["rows"] = _csr(case["n"], case["cols"], r, c, torch.randn(r.numel(), device="cuda", generator=g)), r
        d["x"] = torch.randn(case["cols"], case["k"], device="cuda", generator=g)
        return d
    d["csr"], d["rows"] = _square(case, seed)
    if case["path"] in ("spmv", "build"):
        d["x"] = torch.rand(case["n"], device="cuda", generator=g)
    elif case["path"] == "rwr":
        nodes = _linked(d["csr"], 1)
        d["seeds"] = [int(v) for v in _pick(nodes, case["k"], g).cpu()]
        while len(d["seeds"]) < case["k"]:
            d["seeds"].append(d["seeds"][0])
    elif case["path"] == "diff":
        nodes = _linked(d["csr"], 8)
        d["seed"] = int(_pick(nodes, 1, g)[0])
        d["targets"] = _pick(nodes, case["targets"], g)
        d["feats"] = torch.randn(d["rows"].numel(), case["features"], device="cuda", generator=g)
        d["theta"] = 0.3 * torch.randn(case["features"], generator=torch.Generator().manual_seed(int(seed)))
    return d


def prepare(case, seed):
    if case["path"] == "multi":
        got = [(TiledMatrix(DeviceCsr(csr)), s) for csr, _, s in _graphs(case, seed)]
        return {"case": case, "mats": [m for m, _ in got], "seeds": [s for _, s in got]}
    s = {"case": case, **_inputs(case, seed)}
    if case["path"] == "diff":
        n, _, rp, col, _ = s["csr"]
        s["model"] = EdgeWeightedRWR((n, n, rp, col), s["feats"], s["seed"], DAMP, case["iters"], every=case["every"])
    else:
        s["A"] = DeviceCsr(s["csr"])
        if case["path"] not in ("build", "job"):
            s["M"] = TiledMatrix(s["A"], **FORMATS[case["format"]])
    del s["rows"], s["csr"]
    return s


# ---- one pass

def run(s):
    case = s["case"]
    path = case["path"]
    if path == "spmv":
        return s["M"].spmv(s["x"])
    if path == "spmm":
        return s["M"].spmm(s["x"])
    if path == "build":
        with TiledMatrix(s["A"], **FORMATS[case["format"]]) as M:
            return M.spmv(s["x"])
    if path == "job":
        with TiledMatrix(s["A"], **FORMATS[case["format"]]) as M:
            return M.pagerank(DAMP, 0.0, case["iters"])[0]
    if path == "pagerank":
        p, it, _ = s["M"].pagerank(DAMP, case["tol"], 1000, case["check"])
        return {"p": p, "iters": it}
    if path == "hits":
        a, h, it, _ = s["M"].hits(0.0, case["iters"])
        return {"authorities": a, "hubs": h, "iters": it}
    if path == "rwr":
        r, it, _ = s["M"].rwr(s["seeds"], DAMP, case["tol"], 1000, case["check"])
        return {"r": r, "iters": it}
    if path == "multi":
        return rwr_multi(s["mats"], s["seeds"], DAMP, 0.0, case["iters"], case["iters"])[0]
    theta = s["theta"].clone().requires_grad_()
    scores = s["model"].scores(theta)
    loss = -torch.log(scores[s["targets"]]).sum()
    loss.backward()
    return {"scores": scores.detach(), "grad": theta.grad}


# ---- work and exact values

def work(case):
    """Bytes and operations of one pass: the matrix (8 bytes an entry) and the vectors, once per product."""
    if case["path"] == "multi":
        mid = 2.0 ** ((case["lo"] + case["hi"]) / 2)
        n, nnz, passes, k = case["graphs"] * mid, case["graphs"] * mid * 36, case["iters"], 1
        return {"bytes": passes * (8 * nnz + 8 * n), "flops": passes * 2 * nnz}
    rows = cols = case["n"]
    nnz, k = case["draws"], case.get("k", 1)
    if case["path"] == "spmm":
        cols = case["cols"]
    if case["path"] == "hits":
        rows, cols, nnz = 2 * rows, 2 * cols, 2 * nnz
    if case["path"] in ("rwr", "diff"):
        nnz = 2 * nnz
    once = {"bytes": 8 * nnz + 4 * k * (rows + cols), "flops": 2 * nnz * k}
    passes = case.get("iters", 20 if "tol" in case else 1)
    if case["path"] == "diff":  # forward, adjoint, and the features and the entries' sums
        extra = nnz * (8 * case["features"] + 16)
        return {"bytes": 2 * passes * once["bytes"] + extra, "flops": (4 * passes + 2 * passes) * nnz}
    more = 16 * nnz if case["path"] in ("build", "job") else 0  # the input read and the format written
    return {"bytes": passes * once["bytes"] + more, "flops": passes * once["flops"]}


def _matrix(rp, col, val, shape):
    return torch.sparse_csr_tensor(rp.to(torch.int32), col.to(torch.int32), val, size=shape)


def _walk(A, seeds, tol, check, iters):
    n = A.shape[0]
    e = torch.zeros(n, len(seeds), dtype=torch.float64, device="cuda")
    e[torch.tensor(seeds, device="cuda"), torch.arange(len(seeds), device="cuda")] = 1.0
    r = e
    for it in range(1, iters + 1):
        new = C64 * (A @ r) + (1 - C64) * e
        off = (new - r).abs().sum(0).max()
        r = new
        if tol > 0 and it % check == 0 and float(off) <= tol:
            break
    return r, it


def exact(case, seed):
    """run()'s outputs in 64 bits, from the same 32-bit inputs."""
    path = case["path"]
    if path == "multi":
        return [_walk(_matrix(csr[2], csr[3], csr[4].double(), csr[:2]), [s], 0.0, 1, case["iters"])[0][:, 0]
                for csr, _, s in _graphs(case, seed)]
    d = _inputs(case, seed)
    n, cols, rp, col, val = d["csr"]
    A, rows, col = _matrix(rp, col, val.double(), (n, cols)), d["rows"], col.long()
    if path in ("spmv", "build", "spmm"):
        return A @ d["x"].double()
    if path in ("pagerank", "job"):
        empty = torch.bincount(col, minlength=n) == 0
        p = torch.full((n,), 1.0 / n, dtype=torch.float64, device="cuda")
        for it in range(1, case.get("iters", 1000) + 1):
            new = C64 * (A @ p + p[empty].sum() / n) + (1 - C64) / n
            off = (new - p).abs().sum()
            p = new
            if "tol" in case and it % case["check"] == 0 and float(off) <= case["tol"]:
                break
        return p if path == "job" else {"p": p, "iters": None}
    if path == "hits":
        x = torch.full((n,), 2.0 / n, dtype=torch.float64, device="cuda")
        for _ in range(case["iters"]):
            x = A @ x
            x = torch.cat([x[:n // 2] / x[:n // 2].sum(), x[n // 2:] / x[n // 2:].sum()])
        return {"authorities": x[:n // 2], "hubs": x[n // 2:], "iters": None}
    if path == "rwr":
        return {"r": _walk(A, d["seeds"], case["tol"], case["check"], 1000)[0], "iters": None}
    theta, feats = d["theta"].double().cuda(), d["feats"].double()
    z = feats @ theta
    w = torch.nn.functional.softplus(z)
    total = torch.zeros(n, dtype=torch.float64, device="cuda").index_add_(0, col, w)
    W = w / total[col]
    A = _matrix(rp, col, W, (n, n))
    order = torch.argsort(col, stable=True)
    rpT = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rpT[1:] = torch.cumsum(torch.bincount(col, minlength=n), 0)
    AT = _matrix(rpT, rows[order], W[order], (n, n))
    e = torch.zeros(n, dtype=torch.float64, device="cuda")
    e[d["seed"]] = 1.0
    kept = [e]
    for _ in range(case["iters"]):
        kept.append(C64 * (A @ kept[-1]) + (1 - C64) * e)
    adj = torch.zeros_like(e).index_add_(0, d["targets"], -1.0 / kept[-1][d["targets"]])
    dW = torch.zeros_like(W)
    for r in reversed(kept[:-1]):
        dW += C64 * adj[rows] * r[col]
        adj = C64 * (AT @ adj)
    mean = torch.zeros_like(total).index_add_(0, col, dW * W)
    dz = (dW - mean[col]) / total[col] * torch.sigmoid(z)
    return {"scores": kept[-1], "grad": feats.T @ dz}
