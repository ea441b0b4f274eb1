"""Performance cases of the trace estimator: what a user's program has it do.

Each case is one call (or the pair "make the operator, estimate") through the
public binding, at the sizes of this repository's own workloads or in their
ranges:

* ``estimate``  multilevel log-determinant of a shifted 2D / 3D Laplacian (CSR)
* ``moments``   the moment table itself, for programs that combine it themselves
* ``estrada``   tr exp(A) of a power-law graph (pattern CSR, long rows)
* ``bounds``    the spectral interval of such a graph, the step before it
* ``triangles`` the exact integer triangle moments of such a graph
* ``batch``     the Estrada index of many graphs in one call
* ``dense``     moments of a dense SPD matrix in each arithmetic
* ``nuclear``   tr sqrt(X^T X) of a dense X: with ``form`` the call on a new X
                (Gram matrix formed, one estimate), without it an estimate on
                an operator that the program keeps
* ``sparse_gram``  tr sqrt(X^T X) of a sparse rectangular X, matrix-free

``listed`` gives the named cases, ``draw`` others of the same ranges.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2103_10516_amd import mlct

DEV = "cuda:0"
PREC = {"fp64": mlct.MLCT_FP64, "fp32": mlct.MLCT_FP32, "bf16x3": mlct.MLCT_BF16X3}
MODE = {"direct": mlct.MLCT_DIRECT, "doubling": mlct.MLCT_DOUBLING}


def _levels(text):
    """"8:96,40:32" -> ([8, 40], [96, 32]): degrees and probes of the levels."""
    pairs = [p.split(":") for p in text.split(",")]
    return [int(p[0]) for p in pairs], [int(p[1]) for p in pairs]


def _text(degrees, m):
    return ",".join("%d:%d" % p for p in zip(degrees, m))


def listed():
    return [
        # the smallest use: a two-level estimate of a 1,024-row operator in
        # full precision; launches and latency are all of it
        {"name": "logdet_2d_32_fp64", "kind": "estimate", "dim": 2, "n": 32, "prec": "fp64",
         "mode": "doubling", "levels": "8:96,40:32"},
        # the smallest operator of the 3D Laplacian family, one size off the
        # power of two, at the levels that family uses
        {"name": "logdet_3d_33_fp32", "kind": "estimate", "dim": 3, "n": 33, "prec": "fp32",
         "mode": "doubling", "levels": "8:128,256:64"},
        # the benchmark's own workload
        {"name": "logdet_2d_2048_fp32", "kind": "estimate", "dim": 2, "n": 2048, "prec": "fp32",
         "mode": "doubling", "levels": "25:384,100:64,400:64"},
        # full precision, direct form, an odd grid and a last probe block
        # that is not full
        {"name": "moments_3d_101_fp64", "kind": "moments", "dim": 3, "n": 101, "prec": "fp64",
         "mode": "direct", "degree": 30, "m": 100},
        # Estrada index of the million-vertex power-law graph
        {"name": "estrada_1e6", "kind": "estrada", "d": 1000000, "levels": "10:768,30:192,60:64"},
        # its spectral interval
        {"name": "bounds_1e6", "kind": "bounds", "d": 1000000, "steps": 64},
        # its triangle count
        {"name": "triangles_1e6", "kind": "triangles", "d": 1000000, "m": 1024},
        # the family of 64 graphs of 2,048 to 65,536 vertices in one call
        {"name": "estrada_batch_64", "kind": "batch", "count": 64, "d0": 2048, "ratio": 32.0,
         "levels": "10:768,30:192,60:64"},
        # the dense SPD log-det configuration: small enough for latency
        {"name": "dense_512_fp64", "kind": "dense", "d": 512, "prec": "fp64", "mode": "doubling",
         "degree": 64, "m": 256},
        # nuclear norm of a new dense X in single precision: Gram matrix and
        # one estimate
        {"name": "nuclear_4096_fp32", "kind": "nuclear", "rows": 8192, "cols": 4096,
         "prec": "fp32", "form": True, "levels": "16:3712,64:320,256:64"},
        # the same estimate in split bf16 on an operator that is kept
        {"name": "nuclear_4096_bf16x3", "kind": "nuclear", "rows": 8192, "cols": 4096,
         "prec": "bf16x3", "form": False, "levels": "16:3712,64:320,256:64"},
        # nuclear norm of a sparse rectangular X, two products per step
        {"name": "sparse_gram_1m", "kind": "sparse_gram", "rows": 1 << 20, "cols": 1 << 19,
         "per_row": 8, "degree": 64, "m": 128},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["estimate", "estimate", "moments", "estrada", "bounds", "triangles",
                       "batch", "dense", "dense", "nuclear", "sparse_gram"])
    while True:
        c = _draw(rng, kind)
        if _cost(c) <= 0.9 * _cost(listed()[2]):
            return c


def _draw(rng, kind):
    if kind in ("estimate", "moments"):
        dim = rng.choice([2, 3])
        n = _log_int(rng, 24, 2048) if dim == 2 else _log_int(rng, 10, 128)
        c = {"kind": kind, "dim": dim, "n": n, "prec": rng.choice(["fp32", "fp32", "fp64"]),
             "mode": rng.choice(["doubling", "doubling", "direct"])}
        if kind == "moments":
            c["degree"], c["m"] = _log_int(rng, 4, 200), _log_int(rng, 1, 256)
        else:
            lo = rng.randint(4, 30)
            c["levels"] = _text([lo, lo + _log_int(rng, 10, 300)],
                                [_log_int(rng, 64, 512), _log_int(rng, 16, 128)])
        return c
    if kind == "estrada":
        lo = rng.randint(6, 12)
        return {"kind": kind, "d": _log_int(rng, 1000, 1000000),
                "levels": _text([lo, 3 * lo, 6 * lo], [_log_int(rng, 64, 768),
                                                      _log_int(rng, 32, 192), 64])}
    if kind == "bounds":
        return {"kind": kind, "d": _log_int(rng, 1000, 1000000), "steps": rng.randint(20, 64)}
    if kind == "triangles":
        return {"kind": kind, "d": _log_int(rng, 1000, 1000000), "m": _log_int(rng, 16, 1024)}
    if kind == "batch":
        return {"kind": kind, "count": rng.randint(4, 48), "d0": _log_int(rng, 512, 4096),
                "ratio": round(rng.uniform(1.0, 16.0), 2), "levels": "10:%d,30:%d" % (
                    _log_int(rng, 64, 512), _log_int(rng, 32, 128))}
    if kind == "dense":
        return {"kind": kind, "d": _log_int(rng, 48, 4096),
                "prec": rng.choice(["fp64", "fp32", "bf16x3"]),
                "mode": rng.choice(["doubling", "direct"]), "degree": _log_int(rng, 8, 64),
                "m": _log_int(rng, 16, 1024)}
    if kind == "nuclear":
        cols = _log_int(rng, 128, 4096)
        return {"kind": kind, "rows": cols * 2 - rng.randint(0, 7), "cols": cols,
                "prec": rng.choice(["fp32", "bf16x3"]), "form": rng.random() < 0.5,
                "levels": _text([16, 64], [_log_int(rng, 256, 4096), _log_int(rng, 32, 320)])}
    cols = _log_int(rng, 2000, 500000)
    return {"kind": kind, "rows": int(cols * rng.uniform(0.7, 2.5)), "cols": cols,
            "per_row": rng.randint(3, 12), "degree": rng.randint(8, 64),
            "m": _log_int(rng, 16, 128)}


# ---- inputs -----------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _shift(seed):
    """The Laplacians' diagonal shift: about 0.01, another for each seed."""
    return 0.01 * (1.0 + (seed * 0.6180339887498949) % 1.0)


def _grid_csr(dim, n, seed):
    """5- or 7-point Dirichlet Laplacian + shift I, columns sorted in a row."""
    d = n ** dim
    idx = torch.arange(d, device=DEV, dtype=torch.int64)
    strides = [n ** k for k in reversed(range(dim))]
    cols, keep, vals = [], [], []
    for sign in (-1, 1):
        for st in strides if sign < 0 else reversed(strides):
            pos = (idx // st) % n
            keep.append((pos > 0) if sign < 0 else (pos < n - 1))
            cols.append(idx + sign * st)
            vals.append(-1.0)
        if sign < 0:
            keep.append(torch.ones_like(idx, dtype=torch.bool))
            cols.append(idx)
            vals.append(2.0 * dim + _shift(seed))
    keep = torch.stack(keep, 1)
    col = torch.stack(cols, 1)[keep].to(torch.int32)
    val = torch.tensor(vals, device=DEV, dtype=torch.float32).expand(d, -1)[keep].contiguous()
    rowptr = torch.zeros(d + 1, device=DEV, dtype=torch.int64)
    rowptr[1:] = torch.cumsum(keep.sum(1), 0)
    return rowptr.to(torch.int32), col, val


def _grid_interval(dim, seed):
    s = _shift(seed)
    return 0.99 * s, 4.0 * dim + 1.01 * s


def _graph(d, seed):
    """Chung-Lu power-law graph (average degree 16, exponent 2.5), 0/1 CSR."""
    w = torch.arange(1, d + 1, device=DEV, dtype=torch.float64) ** (-1.0 / 1.5)
    cdf = torch.cumsum(w, 0)
    cdf = cdf / cdf[-1].clone()
    g = _gen(seed)
    e = 8 * d
    u, v = (torch.searchsorted(cdf, torch.rand(e, generator=g, device=DEV, dtype=torch.float64),
                               right=True).clamp_(max=d - 1) for _ in range(2))
    u, v = u[u != v], v[u != v]
    key = torch.unique(torch.cat([u * d + v, v * d + u]))
    row = torch.div(key, d, rounding_mode="floor")
    rowptr = torch.zeros(d + 1, device=DEV, dtype=torch.int64)
    rowptr[1:] = torch.cumsum(torch.bincount(row, minlength=d), 0)
    return rowptr.to(torch.int32), (key - row * d).to(torch.int32)


def _graph_interval(rowptr, col):
    """[-b, b] with b a little above the largest eigenvalue (power steps)."""
    p, c = rowptr.long(), col.long()
    x = torch.ones(p.numel() - 1, device=DEV, dtype=torch.float64)
    lam = torch.ones((), device=DEV, dtype=torch.float64)
    for _ in range(24):
        s = torch.zeros(c.numel() + 1, device=DEV, dtype=torch.float64)
        s[1:] = torch.cumsum(x[c], 0)
        y = s[p[1:]] - s[p[:-1]]
        lam = y.norm() / x.norm()
        x = y / y.norm()
    b = float(math.ceil(1.05 * float(lam) + 1.0))
    return -b, b


def _dense_matrix(case, seed):
    """Dense SPD matrix with eigenvalues in [0.1, 1]: a diagonal spectrum
    under a few random reflections."""
    d = case["d"]
    g = _gen(seed)
    lam = 0.1 + 0.9 * torch.rand(d, generator=g, device=DEV, dtype=torch.float64)
    A = torch.diag(lam)
    for _ in range(8):
        v = torch.randn(d, 1, generator=g, device=DEV, dtype=torch.float64)
        v = v / v.norm()
        Av = A @ v
        A = A - 2 * v @ Av.T - 2 * Av @ v.T + 4 * (v.T @ Av) * (v @ v.T)
    A = 0.5 * (A + A.T)
    return (A if case["prec"] == "fp64" else A.float()).contiguous()


def _dense_x(rows, cols, seed):
    """X = G diag(i^-0.7) V^T / sqrt(rows), FP32: Gaussian G (orthonormal
    columns but for sampling), V a few reflections."""
    g = _gen(seed)
    X = torch.randn(rows, cols, generator=g, device=DEV, dtype=torch.float32)
    X *= torch.arange(1, cols + 1, device=DEV, dtype=torch.float32) ** -0.7 / rows ** 0.5
    for _ in range(8):
        v = torch.randn(cols, 1, generator=g, device=DEV, dtype=torch.float32)
        v = v / v.norm()
        X -= 2 * (X @ v) @ v.T
    return X


def _sparse_x(case, seed):
    """per_row entries in every row, one in each of per_row column bands."""
    rows, cols, k = case["rows"], case["cols"], case["per_row"]
    g = _gen(seed)
    band = cols // k
    col = torch.randint(0, band, (rows, k), generator=g, device=DEV)
    col = (col + band * torch.arange(k, device=DEV)).to(torch.int32).reshape(-1)
    val = torch.randn(rows * k, generator=g, device=DEV)
    rowptr = (torch.arange(rows + 1, device=DEV) * k).to(torch.int32)
    return rowptr, col, val


# sum_j over N(0,1) rows: the squared singular values lie below rows-dependent
# edges; this bound holds for the banded random X above
def _sparse_x_interval(case):
    k, ratio = case["per_row"], case["rows"] / case["cols"]
    return 1e-3, 4.0 * (math.sqrt(k) + math.sqrt(k * ratio)) ** 2 + 60.0


NUCLEAR_INTERVAL = (0.0, 1.5)


def _batch_sizes(case):
    n = max(case["count"] - 1, 1)
    return [int(round(case["d0"] * case["ratio"] ** (i / n))) for i in range(case["count"])]


# ---- the calls ----------------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    ctx = mlct.mlct_create(0)
    st = {"case": case, "ctx": ctx, "seed": 1000 + seed}
    if kind in ("estimate", "moments"):
        st["op"] = mlct.mlct_op_csr(ctx, *_grid_csr(case["dim"], case["n"], seed))
        st["ab"] = _grid_interval(case["dim"], seed)
    elif kind in ("estrada", "bounds", "triangles"):
        g = _graph(case["d"], seed)
        st["op"] = mlct.mlct_op_csr(ctx, *g)
        if kind == "estrada":
            st["ab"] = _graph_interval(*g)
    elif kind == "batch":
        st["items"] = []
        deg, m = _levels(case["levels"])
        for i, d in enumerate(_batch_sizes(case)):
            g = _graph(d, seed + 977 * i)
            a, b = _graph_interval(*g)
            st["items"].append(dict(op=mlct.mlct_op_csr(ctx, *g), kind=mlct.MLCT_EXP, a=a, b=b,
                                    degrees=deg, m=m, seed=st["seed"] + i))
    elif kind == "dense":
        st["op"] = mlct.mlct_op_dense(ctx, _dense_matrix(case, seed))
        st["ab"] = (0.09, 1.01)
    elif kind == "nuclear":
        st["X"] = _dense_x(case["rows"], case["cols"], seed)
        if not case["form"]:
            st["op"] = mlct.mlct_op_gram(ctx, st["X"])
    else:
        st["op"] = mlct.mlct_op_gram_csr(ctx, *_sparse_x(case, seed), case["cols"])
        st["ab"] = _sparse_x_interval(case)
    return st


def _result(r, dtype):
    """An estimate's numbers, the floating ones at ``dtype``."""
    keys = ("estimate", "value", "est_var", "level_mean", "level_var")
    out = {k: np.asarray(r[k], dtype=dtype) for k in keys}
    out["matvecs"] = r["matvecs"]
    out["probe_degrees"] = r["probe_degrees"]
    return out


def _dtype(case):
    """Dense products in single precision or split bf16 give results of FP32
    accuracy, and a program keeps them at that; sparse ones are kept as the
    library returns them."""
    dense = case["kind"] in ("dense", "nuclear")
    return np.float32 if dense and case["prec"] != "fp64" else np.float64


def run(st):
    case, ctx, seed = st["case"], st["ctx"], st["seed"]
    kind = case["kind"]
    if kind == "estimate":
        deg, m = _levels(case["levels"])
        r = mlct.mlct_estimate(ctx, st["op"], mlct.MLCT_LOG, *st["ab"], deg, m, seed,
                               PREC[case["prec"]], MODE[case["mode"]])
        return _result(r, _dtype(case))
    if kind in ("moments", "dense"):
        mu = mlct.mlct_moments(ctx, st["op"], *st["ab"], case["degree"],
                               mlct.rademacher_probes(seed, case["m"]), PREC[case["prec"]],
                               MODE[case["mode"]])
        return {"mu": mu.astype(_dtype(case), copy=False)}
    if kind == "estrada":
        deg, m = _levels(case["levels"])
        r = mlct.mlct_estimate(ctx, st["op"], mlct.MLCT_EXP, *st["ab"], deg, m, seed,
                               mlct.MLCT_FP32, mlct.MLCT_DOUBLING)
        return _result(r, _dtype(case))
    if kind == "bounds":
        return {"ab": np.array(mlct.mlct_bounds(ctx, st["op"], case["steps"], seed, 0.01))}
    if kind == "triangles":
        r, w = mlct.mlct_triangles(ctx, st["op"], case["m"], seed)
        return {"w": w, "sum_w3": r["sum_w3"], "estimate": np.float64(r["estimate"]),
                "estimate_cv": np.float64(r["estimate_cv"]), "a1": np.float64(r["a1"]),
                "a2": np.float64(r["a2"])}
    if kind == "batch":
        rs = mlct.mlct_estimate_batch(ctx, st["items"], mlct.MLCT_FP32, mlct.MLCT_DOUBLING)
        rs = [_result(r, _dtype(case)) for r in rs]
        return {k: np.stack([np.asarray(r[k]) for r in rs]) for k in rs[0]}
    if kind == "nuclear":
        deg, m = _levels(case["levels"])
        op = mlct.mlct_op_gram(ctx, st["X"]) if case["form"] else st["op"]
        r = mlct.mlct_estimate(ctx, op, mlct.MLCT_SQRT, *NUCLEAR_INTERVAL, deg, m, seed,
                               PREC[case["prec"]], mlct.MLCT_DOUBLING)
        if case["form"]:
            op.close()
        return _result(r, _dtype(case))
    r = mlct.mlct_estimate(ctx, st["op"], mlct.MLCT_SQRT, *st["ab"], [case["degree"]],
                           [case["m"]], seed, mlct.MLCT_FP32, mlct.MLCT_DOUBLING)
    return _result(r, _dtype(case))


# ---- work ---------------------------------------------------------------------
def _steps(case):
    """(probes, steps) of each level: a step is one product with A."""
    if "levels" in case:
        pairs = list(zip(*_levels(case["levels"])))
    else:
        pairs = [(case["degree"], case["m"])]
    half = case.get("mode", "doubling") == "doubling"
    return [(m, (n + 1) // 2 if half else n) for n, m in pairs]


def _graph_nnz(d):
    return 15.0 * d  # 16 d less the loops and repeated edges


def work(case):
    """Sparse recurrences: per step the matrix once for up to 64 probes, and
    of the probe vectors V_k and V_{k-1} read and V_{k+1} written.  Dense
    ones: the matrix once, the vectors of each step, 2 d^2 flops per product."""
    kind = case["kind"]
    if kind == "bounds":
        d, k = case["d"], case["steps"]
        # twice through the basis and back for each step's orthogonalisation,
        # of which one reading serves both uses
        return {"bytes": k * 4.0 * _graph_nnz(d) + 2 * 8.0 * d * k * (k + 1) / 2,
                "flops": 2.0 * k * _graph_nnz(d) + 8.0 * d * k * (k + 1) / 2}
    if kind == "triangles":
        d, m = case["d"], case["m"]
        return {"bytes": -(-m // 64) * (2 * 4.0 * _graph_nnz(d)) + m * d * (0.25 + 3 * 2.0),
                "flops": 2 * 2.0 * _graph_nnz(d) * m}
    if kind == "batch":
        one = [_csr_work(d, 4.0 * _graph_nnz(d), _graph_nnz(d), 4, case)
               for d in _batch_sizes(case)]
        return {k: sum(w[k] for w in one) for k in one[0]}
    if kind == "estrada":
        d = case["d"]
        return _csr_work(d, 4.0 * _graph_nnz(d), _graph_nnz(d), 4, case)
    if kind in ("estimate", "moments"):
        d = case["n"] ** case["dim"]
        nnz = (2 * case["dim"] + 1.0) * d
        return _csr_work(d, 8.0 * nnz, nnz, 8 if case["prec"] == "fp64" else 4, case)
    if kind == "sparse_gram":
        nnz = float(case["rows"] * case["per_row"])
        w = _csr_work(case["cols"], 16.0 * nnz, 2 * nnz, 4, case)
        w["bytes"] += sum(m * s for m, s in _steps(case)) * 8.0 * case["rows"]
        return w
    size = 8 if case["prec"] == "fp64" else 4
    d = case["d"] if kind == "dense" else case["cols"]
    products = sum(m * s for m, s in _steps(case))
    w = {"bytes": size * (float(d) * d + 3.0 * d * products), "flops": 2.0 * d * d * products}
    if kind == "nuclear" and case["form"]:
        w["bytes"] += 4.0 * case["rows"] * d
        w["flops"] += float(case["rows"]) * d * d
    return w


def _csr_work(d, matrix_bytes, nnz, size, case):
    passes = sum(-(-m // 64) * s for m, s in _steps(case))
    products = sum(m * s for m, s in _steps(case))
    return {"bytes": passes * (matrix_bytes + 4.0 * d) + products * 3.0 * size * d,
            "flops": products * (2.0 * nnz + 7.0 * d)}


def _cost(case):
    """Rough microseconds, to keep drawn cases below the largest listed one."""
    w = work(case)
    rate = {"batch": 0.5e6, "estrada": 0.9e6, "triangles": 0.5e6, "sparse_gram": 0.8e6}
    flop_rate = 20e6 if case.get("prec") == "fp64" else 60e6
    steps = sum(-(-m // 64) * s for m, s in _steps(case)) if "steps" not in case and \
        case["kind"] != "triangles" else 0
    return w["bytes"] / rate.get(case["kind"], 4e6) + w["flops"] / flop_rate + 4.0 * steps


# ---- the same in 64 bits --------------------------------------------------------
def _mix(x):
    def shr(v, k):  # logical shift of int64
        return (v >> k) & ((1 << (64 - k)) - 1)

    def signed(c):
        return c - (1 << 64) if c >= 1 << 63 else c

    x = (x ^ shr(x, 30)) * signed(0xBF58476D1CE4E5B9)
    x = (x ^ shr(x, 27)) * signed(0x94D049BB133111EB)
    return x ^ shr(x, 31)


def _probes(d, seed, first, count):
    """Rademacher probes first .. first + count - 1 of the seed, d x count:
    counter-based SplitMix64, one word of signs per 64 rows."""
    gamma = 0x9E3779B97F4A7C15 - (1 << 64)
    ids = torch.arange(first + 1, first + count + 1, device=DEV, dtype=torch.int64)
    key = _mix(seed + ids * gamma)
    chunk = torch.arange(1, -(-d // 64) + 1, device=DEV, dtype=torch.int64)
    word = _mix(key[None, :] + chunk[:, None] * gamma)
    bit = torch.arange(64, device=DEV, dtype=torch.int64)
    z = 1.0 - 2.0 * ((word[:, None, :] >> bit[None, :, None]) & 1).double()
    return z.reshape(-1, count)[:d].contiguous()


def _mu(apply, z, a, b, n, doubling):
    """Moments z^T T_j(A_hat) z, j = 0..n, of the columns of z."""
    sc, sh = 2.0 / (b - a), -(a + b) / (b - a)

    def hat(v):
        return sc * apply(v) + sh * v

    def dot(u, v):
        return (u * v).sum(0)

    mu = torch.zeros(z.shape[1], n + 1, device=DEV, dtype=torch.float64)
    mu[:, 0] = dot(z, z)
    if n == 0:
        return mu
    v0, v1 = z, hat(z)
    mu[:, 1] = dot(z, v1)
    if not doubling:
        for j in range(2, n + 1):
            v0, v1 = v1, 2 * hat(v1) - v0
            mu[:, j] = dot(z, v1)
        return mu
    for k in range(1, (n + 1) // 2 + 1):  # v1 = T_k z, v0 = T_{k-1} z
        if k > 1:
            mu[:, 2 * k - 1] = 2 * dot(v1, v0) - mu[:, 1]
        if 2 * k <= n:
            mu[:, 2 * k] = 2 * dot(v1, v1) - mu[:, 0]
        if k < (n + 1) // 2:
            v0, v1 = v1, 2 * hat(v1) - v0
    return mu


def _coefficients(f, a, b, n):
    """Interpolant of f on [a, b] at the Chebyshev extreme points."""
    k = np.arange(n + 1)
    t = f(0.5 * (b - a) * np.cos(np.pi * k / n) + 0.5 * (a + b))
    t[0] *= 0.5
    t[-1] *= 0.5
    c = 2.0 / n * (np.cos(np.pi * np.outer(k, k) / n) @ t)
    c[0] *= 0.5
    c[-1] *= 0.5
    return c


def _estimate(apply, d, f, a, b, degrees, m, seed, width=64):
    c = torch.from_numpy(_coefficients(f, a, b, degrees[-1])).to(DEV)
    mean, var, first, low = [], [], 0, 0
    for n, count in zip(degrees, m):
        q = []
        for p in range(0, count, width):
            z = _probes(d, seed, first + p, min(width, count - p))
            mu = _mu(apply, z, a, b, n, True)
            q.append(mu[:, low:n + 1] @ c[low:n + 1])
        q = torch.cat(q)
        mean.append(float(q.mean()))
        var.append(float(q.var()))
        first, low = first + count, n + 1
    value = sum(mean)
    return {"estimate": np.float64(value), "value": np.float64(value),
            "est_var": np.float64(sum(v / k for v, k in zip(var, m))),
            "level_mean": np.array(mean), "level_var": np.array(var), "matvecs": None,
            "probe_degrees": None}


def _grid_apply(dim, n, seed):
    """The Laplacian by shifts of the grid, its diagonal as stored in FP32."""
    diag = float(np.float32(2.0 * dim + _shift(seed)))

    def apply(v):
        g = v.reshape((n,) * dim + (v.shape[1],))
        out = diag * g
        for k in range(dim):
            lo, hi = out.narrow(k, 1, n - 1), out.narrow(k, 0, n - 1)
            lo -= g.narrow(k, 0, n - 1)
            hi -= g.narrow(k, 1, n - 1)
        return out.reshape(v.shape)

    return apply


def _sparse_apply(rowptr, col, val, shape):
    A = torch.sparse_csr_tensor(rowptr.long(), col.long(), val.double(), size=shape)
    return lambda v: A @ v


def _pattern_apply(rowptr, col):
    d = rowptr.numel() - 1
    return _sparse_apply(rowptr, col, torch.ones_like(col, dtype=torch.float64), (d, d))


def _lanczos_interval(apply, d, steps, seed, margin):
    """Extreme Ritz values, widened by their residual bounds and the margin."""
    Q = torch.zeros(steps + 1, d, device=DEV, dtype=torch.float64)
    Q[0] = _probes(d, seed, 0, 1)[:, 0] / math.sqrt(d)
    al, be = [], []
    for j in range(steps):
        w = apply(Q[j][:, None])[:, 0]
        al.append(float(Q[j] @ w))
        for _ in range(2):
            w = w - Q[:j + 1].T @ (Q[:j + 1] @ w)
        be.append(float(w.norm()))
        if be[-1] <= 1e-12 * max(1.0, abs(al[-1])):
            break
        Q[j + 1] = w / be[-1]
    T = np.diag(al) + np.diag(be[:-1], 1) + np.diag(be[:-1], -1)
    th, s = np.linalg.eigh(T)
    w = th[-1] - th[0]
    return np.array([th[0] - abs(be[-1] * s[-1, 0]) - margin * w,
                     th[-1] + abs(be[-1] * s[-1, -1]) + margin * w])


def exact(case, seed):
    kind, pseed = case["kind"], 1000 + seed
    half = case.get("mode", "doubling") == "doubling"
    if kind in ("estimate", "moments"):
        d = case["n"] ** case["dim"]
        apply, ab = _grid_apply(case["dim"], case["n"], seed), _grid_interval(case["dim"], seed)
        if kind == "estimate":
            return _estimate(apply, d, np.log, *ab, *_levels(case["levels"]), pseed)
        mu = [_mu(apply, _probes(d, pseed, p, min(64, case["m"] - p)), *ab, case["degree"], half)
              for p in range(0, case["m"], 64)]
        return {"mu": torch.cat(mu)}
    if kind == "bounds":
        return {"ab": _lanczos_interval(_pattern_apply(*_graph(case["d"], seed)), case["d"],
                                        case["steps"], pseed, 0.01)}
    if kind == "estrada":
        g = _graph(case["d"], seed)
        return _estimate(_pattern_apply(*g), case["d"], np.exp, *_graph_interval(*g),
                         *_levels(case["levels"]), pseed)
    if kind == "triangles":
        apply = _pattern_apply(*_graph(case["d"], seed))
        total = 0.0
        for p in range(0, case["m"], 64):
            y = apply(_probes(case["d"], pseed, p, min(64, case["m"] - p)))
            total += float((y * apply(y)).sum())
        return {"w": None, "sum_w3": None, "estimate": np.float64(total / (6.0 * case["m"])),
                "estimate_cv": None, "a1": None, "a2": None}
    if kind == "batch":
        rs = []
        for i, d in enumerate(_batch_sizes(case)):
            g = _graph(d, seed + 977 * i)
            rs.append(_estimate(_pattern_apply(*g), d, np.exp, *_graph_interval(*g),
                                *_levels(case["levels"]), pseed + i, 256))
        return {k: None if rs[0][k] is None else np.stack([r[k] for r in rs]) for k in rs[0]}
    if kind == "dense":
        A = _dense_matrix(case, seed).double()
        z = _probes(case["d"], pseed, 0, case["m"])
        return {"mu": _mu(lambda v: A @ v, z, 0.09, 1.01, case["degree"], half)}
    if kind == "nuclear":
        X = _dense_x(case["rows"], case["cols"], seed).double()
        G = X.T @ X
        return _estimate(lambda v: G @ v, case["cols"], np.sqrt, *NUCLEAR_INTERVAL,
                         *_levels(case["levels"]), pseed, 4096)
    rowptr, col, val = _sparse_x(case, seed)
    X = _sparse_apply(rowptr, col, val, (case["rows"], case["cols"]))
    row = torch.arange(case["rows"], device=DEV).repeat_interleave(case["per_row"])
    order = torch.argsort(col.long() * case["rows"] + row)
    tptr = torch.zeros(case["cols"] + 1, device=DEV, dtype=torch.int64)
    tptr[1:] = torch.cumsum(torch.bincount(col.long(), minlength=case["cols"]), 0)
    Xt = _sparse_apply(tptr, row[order], val[order], (case["cols"], case["rows"]))
    return _estimate(lambda v: Xt(X(v)), case["cols"], np.sqrt, *_sparse_x_interval(case),
                     [case["degree"]], [case["m"]], pseed)
