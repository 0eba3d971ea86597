"""The cases this library's speed is measured on.

One case is one call of a public entry point as a program makes it: device tensors and a memory
limit in, fresh result tensors out, the workspace taken by the call.  The listed cases are the
workloads of the benchmark (`bench.py`, `workloads.py`) at their own sizes, a search with few
queries as a service makes it, and the double-precision kernel product at a size that a
pass affords.  `draw` gives further calls over the range of sizes, dimensions, metrics and limits
between and around them.

Keys of a case: "op" is "knn", "kmv" or "sgpr"; the others are that entry point's arguments and
"data", the values' distribution.
"""
from __future__ import annotations

import math

import torch

import paper_2206_14148_amd as knn

MB, GB = 10 ** 6, 10 ** 9


def _knn(name, m, n, d, k, data, limit, metric="l2", q_is_x=False):
    return {"name": name, "op": "knn", "m": m, "n": n, "d": d, "k": k, "metric": metric, "data": data,
            "q_is_x": q_is_x, "limit": limit}


def _kmv(name, n, m, d, lengthscale, dtype="f32", z_is_x=True):
    return {"name": name, "op": "kmv", "n": n, "m": m, "d": d, "lengthscale": lengthscale, "dtype": dtype,
            "z_is_x": z_is_x, "limit": 1 * GB}


def _sgpr(name, m, n, d, lengthscale):
    return {"name": name, "op": "sgpr", "m": m, "n": n, "d": d, "lengthscale": lengthscale, "limit": 1 * GB}


def listed():
    return [
        # a service answering a handful of queries against a table of word vectors whose rows
        # are not a multiple of 16 bytes: what counts is how long one answer takes
        _knn("serve_d50", 16, 100_003, 50, 10, "gmm", 256 * MB),
        # the smallest random-data row of the paper's table
        _knn("random_d16", 1_000, 10_000, 16, 10, "normal", 64 * MB),
        # the kNN graph of a point cloud (normal estimation, graph networks)
        _knn("pointcloud_d3", 1_000_000, 1_000_000, 3, 16, "uniform", 1 * GB, q_is_x=True),
        # image vectors: sparse non-negative pixels, long rows
        _knn("images_d784", 10_000, 1_000_000, 784, 10, "sparse", 2 * GB),
        # clustered embeddings, the largest search: the benchmark's default workload
        _knn("embeddings_d128", 100_000, 10_000_000, 128, 100, "gmm", 8 * GB),
        # a limit far below the data's size: the memory-limit sweep's 1 GB entry
        _knn("memlimit_d256", 50_000, 2_000_000, 256, 32, "normal", 1 * GB),
        # word vectors under the cosine distance
        _knn("cosine_d100", 10_000, 1_183_514, 100, 10, "gmm", 1 * GB, metric="cosine"),
        # the L1 rows of the paper's table
        _knn("l1_d100", 10_000, 1_000_000, 100, 10, "normal", 1 * GB, metric="l1"),
        # kernel matrix times vector, one-dimensional inputs: the matrix would take 4 TB
        _kmv("kernel_d1", 1_000_000, 1_000_000, 1, 1.0),
        # the same with several features, on the matrix cores
        _kmv("kernel_d32", 200_000, 200_000, 32, 6.0),
        # and in double precision, the precision the paper evaluates it in; an odd size
        _kmv("kernel_f64_d1", 200_003, 200_003, 1, 1.0, dtype="f64"),
        # the sums of sparse GP regression: 4000 inducing points, two million rows of 11 features
        _sgpr("sgpr_m4000_d11", 4_000, 2_049_280, 11, 3.0),
    ]


def _log(rng, low, high):
    """A whole number between low and high, its logarithm uniform."""
    return int(min(high, max(low, round(math.exp(rng.uniform(math.log(low), math.log(high + 1)))))))


def draw(rng):
    """One more call of the same ranges.  Sizes whose work would exceed the listed cases' are cut."""
    kind = rng.choice(("cloud", "lowd", "mid", "mid", "wide", "cosine", "l1", "kmv", "kmv", "kmv_f64", "sgpr"))
    limit = rng.choice((64 * MB, 256 * MB, 1 * GB, 2 * GB, 8 * GB))
    if kind == "cloud":
        n = _log(rng, 10_000, 1_000_000)
        own = rng.random() < 0.5
        m = n if own else _log(rng, 1_000, 1_000_000)
        return _unnamed(_knn("", m, n, rng.choice((2, 3)), _log(rng, 1, 32), rng.choice(("uniform", "normal")),
                             max(limit, 256 * MB), q_is_x=own))
    if kind == "lowd":
        n = _log(rng, 10_000, 1_000_000)
        m = _log(rng, 1_000, min(1_000_000, 200_000_000_000 // n))
        return _unnamed(_knn("", m, n, rng.randint(4, 8), _log(rng, 1, 32), rng.choice(("uniform", "normal")),
                             max(limit, 256 * MB)))
    if kind == "mid":
        d = _log(rng, 9, 256)
        n = _log(rng, 10_000, min(10_000_000, 1_280_000_000 // d))
        m = _log(rng, 1, max(16, min(100_000, 25_000_000_000_000 // (n * d))))
        return _unnamed(_knn("", m, n, d, _log(rng, 1, 100), rng.choice(("normal", "gmm")), max(limit, 256 * MB)))
    if kind == "wide":
        d = _log(rng, 257, 1_024)
        n = _log(rng, 10_000, 1_000_000)
        m = _log(rng, 1, max(16, min(10_000, 3_000_000_000_000 // (n * d))))
        return _unnamed(_knn("", m, n, d, _log(rng, 1, 32), rng.choice(("normal", "sparse")), max(limit, 256 * MB)))
    if kind == "cosine":
        d = _log(rng, 25, 300)
        n = _log(rng, 10_000, 1_200_000)
        m = _log(rng, 1, 10_000)
        return _unnamed(_knn("", m, n, d, _log(rng, 1, 100), "gmm", max(limit, 256 * MB), metric="cosine"))
    if kind == "l1":
        d = _log(rng, 3, 200)
        n = _log(rng, 10_000, 1_000_000)
        m = _log(rng, 1, max(16, min(10_000, 1_000_000_000_000 // (n * d))))
        return _unnamed(_knn("", m, n, d, _log(rng, 1, 32), rng.choice(("normal", "uniform", "gmm")),
                             max(limit, 256 * MB), metric="l1"))
    if kind == "kmv":
        d = _log(rng, 1, 64)
        most = 1_000_000 if d == 1 else 200_000
        n = _log(rng, 1_000, most)
        m = _log(rng, 1_000, most)
        return _unnamed(_kmv("", n, m, d, round(math.sqrt(d) * rng.uniform(0.3, 1.5), 3), z_is_x=n == m))
    if kind == "kmv_f64":
        d = _log(rng, 1, 12)
        n = _log(rng, 1_000, 200_000)
        m = _log(rng, 1_000, min(200_000, 40_000_000_000 // (n * d)))
        return _unnamed(_kmv("", n, m, d, round(math.sqrt(d) * rng.uniform(0.3, 1.5), 3), dtype="f64", z_is_x=n == m))
    m = _log(rng, 100, 4_000)
    return _unnamed(_sgpr("", m, _log(rng, 10_000, 2_000_000), rng.randint(1, 16), round(rng.uniform(1.0, 4.0), 3)))


def _unnamed(case):
    del case["name"]
    return case


# ---- inputs ---------------------------------------------------------------------------------

_ROWS = 1 << 20  # rows made at a time, bounds the temporaries


def _points(gen, rows, d, data, centres, dtype=torch.float32):
    if data == "uniform":
        return torch.rand(rows, d, generator=gen, device="cuda", dtype=dtype)
    x = torch.randn(rows, d, generator=gen, device="cuda", dtype=dtype)
    for s in range(0, rows, _ROWS):
        e = min(rows, s + _ROWS)
        if data == "sparse":  # an entry is 0 with probability 0.8, else uniform in (0, 1]
            keep = torch.rand(e - s, d, generator=gen, device="cuda") < 0.2
            x[s:e] = torch.where(keep, 1.0 - torch.rand(e - s, d, generator=gen, device="cuda"), 0.0)
        elif data == "gmm":   # a component's centre plus unit noise
            x[s:e] += centres[torch.randint(centres.shape[0], (e - s,), generator=gen, device="cuda")]
    return x


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    d = case["d"]
    if case["op"] == "knn":
        centres = 2.0 * torch.randn(1_000, d, generator=gen, device="cuda")
        X = _points(gen, case["n"], d, case["data"], centres)
        Q = X if case["q_is_x"] else _points(gen, case["m"], d, case["data"], centres)
        return {"case": case, "Q": Q, "X": X}
    if case["op"] == "kmv":
        dtype = torch.float64 if case["dtype"] == "f64" else torch.float32
        X = _points(gen, case["n"], d, "normal", None, dtype)
        Z = X if case["z_is_x"] else _points(gen, case["m"], d, "normal", None, dtype)
        v = torch.randn(case["m"], generator=gen, device="cuda", dtype=dtype)
        return {"case": case, "X": X, "Z": Z, "v": v}
    X = _points(gen, case["n"], d, "normal", None)
    y = torch.randn(case["n"], generator=gen, device="cuda")
    U = X[: case["m"]].clone()  # the usual start: inducing points are the first data points
    return {"case": case, "U": U, "X": X, "y": y}


def run(state):
    c = state["case"]
    if c["op"] == "knn":
        return knn.knn_search(state["Q"], state["X"], c["k"], c["limit"], metric=c["metric"])
    if c["op"] == "kmv":
        return knn.kmv_apply(state["X"], state["Z"], state["v"], 1.0, c["lengthscale"], c["limit"])
    return knn.sgpr_accumulate(state["U"], state["X"], state["y"], 1.0, c["lengthscale"], c["limit"])


# ---- what a pass cannot do without ----------------------------------------------------------

def work(case):
    d = case["d"]
    if case["op"] == "knn":
        m, n, k = case["m"], case["n"], case["k"]
        nbytes = 4 * d * (n + (0 if case["q_is_x"] else m)) + 8 * m * k
        if d <= 3 and case["metric"] == "l2":
            # where points are so few-dimensional a search need not look at every pair: what
            # is left is the evaluation of the winners
            return {"bytes": nbytes, "flops": 3 * d * m * k}
        return {"bytes": nbytes, "flops": 2 * d * m * n}
    if case["op"] == "kmv":
        n, m = case["n"], case["m"]
        size = 8 if case["dtype"] == "f64" else 4
        if d == 1:
            # on a line the entries need not be made one by one: sources that lie close together
            # act through a short series.  What is left is the points themselves
            return {"bytes": size * (n + (0 if case["z_is_x"] else m) + m) + 8 * n, "flops": 5 * (n + m)}
        # per entry the distance, the exponential counted as one operation, and the sum
        return {"bytes": size * (d * (n + (0 if case["z_is_x"] else m)) + m) + 8 * n, "flops": (2 * d + 3) * n * m}
    m, n = case["m"], case["n"]
    # one triangle of the symmetric product, the kernel matrix, the product with y
    return {"bytes": 4 * (d * (m + n) + n) + 8 * (m * m + m), "flops": n * m * (m + 1) + (2 * d + 4) * n * m}


def tolerance(case):
    if case["op"] == "knn":
        # a search gives the same neighbours and the same rounded distances however it is cut
        return "exact"
    if case["op"] == "kmv":
        # against the double-precision entry point on the same numbers 1.7e-7 was seen (max 8e-7), and
        # for that one 2e-14 against sums in the opposite order
        return {"rel": 2e-13, "max": 2e-12} if case["dtype"] == "f64" else {"rel": 8e-7, "max": 1e-5}
    # against double precision 3.4e-8 was seen for A and 1.1e-7 for b
    return {"rel": 5e-7, "max": 5e-6}


# ---- the same in 64 bits --------------------------------------------------------------------

def exact(case, seed):
    """What `run` returns, in double precision from plain torch; None where that takes too long.
    A search's indices have no such value: neighbours that are equally far may come in any order."""
    state = prepare(case, seed)
    if case["op"] == "knn":
        return _exact_knn(case, state["Q"].double(), state["X"].double())
    if case["op"] == "kmv":
        return _exact_kmv(case, state["X"].double(), state["Z"].double(), state["v"].double())
    U, X, y = (state[a].double() for a in ("U", "X", "y"))
    A = torch.zeros(case["m"], case["m"], dtype=torch.float64, device="cuda")
    b = torch.zeros(case["m"], dtype=torch.float64, device="cuda")
    for s in range(0, case["n"], 1 << 17):
        K = _gaussian(U, X[s:s + (1 << 17)], case["lengthscale"])
        A += K @ K.T
        b += K @ y[s:s + (1 << 17)]
    return A, b


def _exact_knn(case, Q, X):
    m, n, d, k = case["m"], case["n"], case["d"], case["k"]
    if m * n > 2e10 or m * n * d > (1e12 if case["metric"] == "l1" else 2e13):
        return None
    dist = torch.empty(m, k, dtype=torch.float64, device="cuda")
    rows = max(1, min(m, (1 << (24 if case["metric"] == "l1" else 29)) // n))
    if case["metric"] == "cosine":
        Q, X = Q / Q.norm(dim=1, keepdim=True), X / X.norm(dim=1, keepdim=True)
    xn, Xt = (X * X).sum(1), X.T.contiguous()
    for s in range(0, m, rows):
        q = Q[s:s + rows]
        if case["metric"] == "l1":
            D = torch.zeros(q.shape[0], n, dtype=torch.float64, device="cuda")
            for t in range(d):
                D += (q[:, t, None] - Xt[None, t]).abs_()
        elif case["metric"] == "cosine":
            D = 1 - q @ X.T
        elif d <= 8:
            D = sum((q[:, t, None] - X[None, :, t]).square_() for t in range(d))
        else:
            D = torch.addmm(xn[None, :] + (q * q).sum(1)[:, None], q, X.T, alpha=-2)
        dist[s:s + rows] = D.topk(k, dim=1, largest=False).values
    return None, dist


def _gaussian(X, Z, lengthscale):
    c = 0.5 / lengthscale ** 2
    if X.shape[1] <= 2:
        return sum((X[:, t, None] - Z[None, :, t]).square_() for t in range(X.shape[1])).mul_(-c).exp_()
    xn, zn = (X * X).sum(1), (Z * Z).sum(1)
    return torch.addmm(xn[:, None] + zn[None, :], X, Z.T, alpha=-2).mul_(-c).exp_()


def _exact_kmv(case, X, Z, v):
    n, m, d = case["n"], case["m"], case["d"]
    if n * m * d > 5e11 and d > 8:
        return None
    y = torch.empty(n, dtype=torch.float64, device="cuda")
    rows = max(1, min(n, (1 << 25) // m))
    for s in range(0, n, rows):
        y[s:s + rows] = _gaussian(X[s:s + rows], Z, case["lengthscale"]) @ v
    return y
