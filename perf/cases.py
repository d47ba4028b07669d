"""Timed cases of the library's main path: the contractions, products and
iterations a program asks of it through the Python binding, from calls where
launches count to ones that fill the GPU.

Each listed case stands for one use; `draw` gives further cases of the same
ranges.  Sizes and distributions are those of the repository's benchmark
workloads and tests (Erdos-Renyi, R-MAT, 27-point stencils, power-law rows,
Bernoulli tensors), generated on the GPU from the seed.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_1512_00066_amd as srtc

DEV = "cuda"
ABCD = (0.57, 0.19, 0.19, 0.05)  # R-MAT level probabilities
NO_PATH = (2 ** 31 - 1) // 2
DTYPES = {"f64": torch.float64, "f32": torch.float32, "i32": torch.int32}
SIZES = {"f64": 8, "f32": 4, "i32": 4}
SEMIRING = {"f64": "plus_times", "f32": "plus_times", "i32": "min_plus"}


def listed():
    return [
        # one small graph product among many calls: the smallest instance
        # of the batched workload, called by itself (latency and launches)
        {"name": "spgemm_er1000_i32", "kind": "spgemm", "graph": "er", "n": 1000, "d": 8.0, "dtype": "i32"},
        # an ordinary sparse product: short rows, hash-sized outputs, odd n
        {"name": "spgemm_er50021_f32", "kind": "spgemm", "graph": "er", "n": 50021, "d": 16.0, "dtype": "f32"},
        # the largest product that returns its output whole: R-MAT 18
        # squared, heavy skewed rows
        {"name": "spgemm_rmat18_f64", "kind": "spgemm", "graph": "rmat", "n": 1 << 18, "d": 16.0, "dtype": "f64"},
        # independent uneven graphs squared in one call
        {"name": "batch20_er_i32", "kind": "batch", "count": 20, "n_lo": 1000, "n_hi": 100000, "d": 18.0,
         "dtype": "i32"},
        # many-source shortest paths and reachability on a skewed graph
        {"name": "paths_rmat18_64src", "kind": "paths", "n": 1 << 18, "d": 16.0, "nsrc": 64},
        # products wanted only at the positions of a mask (triangle shape)
        {"name": "masked_rmat18_f64", "kind": "masked", "n": 1 << 18, "d": 16.0, "dtype": "f64"},
        # all-pairs shortest paths of a complete weighted graph
        {"name": "apsp_dense2000", "kind": "apsp", "n": 2000, "density": 1.0},
        # dense times dense on the matrix cores, aligned and in fp64
        {"name": "gemm_4096_f64", "kind": "gemm", "m": 4096, "n": 4096, "k": 4096, "dtype": "f64"},
        # the same in fp32 with sides that no tile divides
        {"name": "gemm_ragged_f32", "kind": "gemm", "m": 6001, "n": 5003, "k": 7004, "dtype": "f32"},
        # a 1% sparse integral tensor times dense amplitudes (the largest
        # term of the MP3 energy): sparse times wide dense
        {"name": "spmm_amplitudes_f64", "kind": "spmm", "m": 16384, "k": 16384, "d": 163.84, "width": 1024,
         "dtype": "f64"},
        # taking in a graph: index-value pairs with repeats to CSR
        {"name": "fold_rmat20_f32", "kind": "fold", "n": 1 << 20, "d": 16.0, "dtype": "f32"},
        # a linear solve by Jacobi iteration on a 27-point stencil
        {"name": "jacobi_stencil100_f64", "kind": "jacobi", "g": 100, "rel": 1e-6, "dtype": "f64"},
    ]


# ------------------------------------------------------------------ drawing --
def _log(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi]."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    kind = rng.choice(["spgemm", "spgemm", "spgemm", "batch", "paths", "masked", "apsp", "gemm", "gemm", "spmm", "spmm",
                       "fold", "jacobi", "tensor"])
    dt3, dt2 = rng.choice(["f64", "f32", "i32"]), rng.choice(["f64", "f32"])
    if kind == "spgemm":
        graph = rng.choice(["er", "er", "rmat", "stencil", "power"])
        if graph == "er":
            return {"kind": kind, "graph": graph, "n": _log(rng, 200, 100000), "d": round(rng.uniform(2, 24), 2),
                    "dtype": dt3}
        if graph == "rmat":
            return {"kind": kind, "graph": graph, "n": _log(rng, 1000, 1 << 17), "d": round(rng.uniform(4, 16), 2),
                    "dtype": dt3}
        if graph == "stencil":
            return {"kind": kind, "graph": graph, "g": rng.randint(8, 40), "dtype": dt3}
        return {"kind": kind, "graph": graph, "n": _log(rng, 1 << 10, 1 << 15), "gamma": round(rng.uniform(1.8, 2.6), 2),
                "dtype": dt3}
    if kind == "batch":
        return {"kind": kind, "count": rng.randint(2, 20), "n_lo": 1000, "n_hi": _log(rng, 2000, 60000),
                "d": round(rng.uniform(4, 18), 2), "dtype": rng.choice(["i32", "f32"])}
    if kind == "paths":
        return {"kind": kind, "n": _log(rng, 1000, 1 << 18), "d": round(rng.uniform(4, 16), 2),
                "nsrc": rng.choice([1, 4, 8, 13, 32, 50, 64])}
    if kind == "masked":
        return {"kind": kind, "n": _log(rng, 1000, 1 << 18), "d": round(rng.uniform(4, 16), 2), "dtype": dt3}
    if kind == "apsp":
        return {"kind": kind, "n": _log(rng, 64, 2000), "density": rng.choice([1.0, 1.0, 0.2, 0.02])}
    if kind == "gemm":
        return {"kind": kind, "m": _log(rng, 64, 6000), "n": _log(rng, 64, 6000), "k": _log(rng, 64, 6000), "dtype": dt2}
    if kind == "spmm":
        width = rng.choice([1, 2, 7, 8, 16, 32, 50, 64, 100, 128, 256, 1000, 1024])
        m, k = _log(rng, 1000, 200000), _log(rng, 1000, 200000)
        d = rng.uniform(4, 160)
        return {"kind": kind, "m": m, "k": k, "d": round(max(2.0, min(d, 2.5e9 / m / width)), 2), "width": width,
                "dtype": dt3}
    if kind == "fold":
        return {"kind": kind, "n": _log(rng, 1000, 1 << 20), "d": round(rng.uniform(4, 16), 2), "dtype": dt3}
    if kind == "jacobi":
        return {"kind": kind, "g": rng.randint(20, 100), "rel": rng.choice([1e-3, 1e-4]), "dtype": dt2}
    # an order-3 tensor of index-value pairs times a dense matrix
    return {"kind": kind, "i": _log(rng, 64, 640), "j": _log(rng, 64, 640), "k": _log(rng, 64, 640),
            "l": rng.choice([8, 33, 64, 100, 128]), "density": rng.choice([1e-3, 3e-3, 1e-2]), "dtype": dt2}


# ------------------------------------------------------------------- inputs --
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _values(g, count, dtype, lo=1, hi=100):
    if dtype == "i32":
        return torch.randint(lo, hi + 1, (count,), generator=g, device=DEV, dtype=torch.int32)
    # (0, 1]: a stored 0 is no entry, and outputs would lose a few by the seed
    return 1 - torch.rand(count, generator=g, device=DEV, dtype=DTYPES[dtype])


def _base():
    """Random graphs come from one fixed stream and are then relabelled and
    given values by the seed: another seed is another matrix, with as many
    entries, products and outputs, so outputs of different seeds have the
    same size."""
    return _gen(151200066)


def _relabelled(g, r, c, n):
    """The pairs with the n vertices renamed at random."""
    p = torch.randperm(n, generator=g, device=DEV)
    return p[r], p[c]


def _er_keys(g, n, d):
    """About n d distinct off-diagonal positions of an n x n matrix, sorted."""
    k = torch.randint(0, n * n, (int(n * d),), generator=_base(), device=DEV)
    k = k[k // n != k % n]
    r, c = _relabelled(g, k // n, k % n, n)
    return torch.unique(r * n + c)


def _rmat_pairs(g, n, d):
    """About n d pairs (row, column) of an R-MAT graph on 2^s >= n relabelled
    vertices, those inside n x n kept; repeats and self-loops stay."""
    s = max(1, (n - 1).bit_length())
    full = 1 << s
    e = int(full * d)
    r = torch.zeros(e, dtype=torch.int64, device=DEV)
    c = torch.zeros(e, dtype=torch.int64, device=DEV)
    a, b, cc, _ = ABCD
    base = _base()
    for _ in range(s):
        u = torch.rand(e, generator=base, device=DEV)
        rb = (u >= a + b).long()
        cb = (((u >= a) & (u < a + b)) | (u >= a + b + cc)).long()
        r = 2 * r + rb
        c = 2 * c + cb
    if full != n:
        r, c = _relabelled(base, r, c, full)
        keep = (r < n) & (c < n)
        r, c = r[keep], c[keep]
    return _relabelled(g, r, c, n)


def _rmat_keys(g, n, d):
    r, c = _rmat_pairs(g, n, d)
    return torch.unique(r * n + c)


def _stencil(gs):
    """CSR pattern of the 27-point stencil on a gs^3 grid: (rowptr, col)."""
    n = gs ** 3
    i = torch.arange(n, device=DEV)
    z, y, x = i // (gs * gs), (i // gs) % gs, i % gs
    cols = torch.empty((n, 27), dtype=torch.int32, device=DEV)
    ok = torch.empty((n, 27), dtype=torch.bool, device=DEV)
    q = 0
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                zz, yy, xx = z + dz, y + dy, x + dx
                ok[:, q] = (zz >= 0) & (zz < gs) & (yy >= 0) & (yy < gs) & (xx >= 0) & (xx < gs)
                cols[:, q] = ((zz * gs + yy) * gs + xx).int()
                q += 1
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rowptr[1:] = torch.cumsum(ok.sum(1), 0)
    return rowptr, cols[ok]


def _power_cdf(n, gamma):
    w = np.arange(1, n + 1, dtype=np.float64) ** (-gamma)
    return w / w.sum()


def _power_keys(g, n, gamma):
    """Rows whose lengths follow k^-gamma for k in 1..n, uniform columns."""
    cdf = torch.as_tensor(np.cumsum(_power_cdf(n, gamma)), device=DEV)
    base = _base()
    u = torch.rand(n, generator=base, device=DEV, dtype=torch.float64)
    deg = torch.clamp(torch.searchsorted(cdf, u, right=True) + 1, max=n)
    rows = torch.repeat_interleave(torch.arange(n, device=DEV), deg)
    r, c = _relabelled(g, rows, torch.randint(0, n, (rows.numel(),), generator=base, device=DEV), n)
    return torch.unique(r * n + c)


def _csr(keys, m, n, val):
    """The library's CSR of sorted distinct keys row * n + column."""
    rowptr = torch.zeros(m + 1, dtype=torch.int64, device=DEV)
    rowptr[1:] = torch.cumsum(torch.bincount(keys // n, minlength=m), 0)
    return srtc.CSR(rowptr, (keys % n).int(), val, (m, n))


def _graph(case, g):
    graph, dt = case.get("graph", "rmat"), case.get("dtype", "i32")
    if graph == "stencil":
        rowptr, col = _stencil(case["g"])
        return srtc.CSR(rowptr, col, _values(g, col.numel(), dt), (case["g"] ** 3,) * 2)
    n = case["n"]
    if graph == "er":
        keys = _er_keys(g, n, case["d"])
    elif graph == "rmat":
        keys = _rmat_keys(g, n, case["d"])
    else:
        keys = _power_keys(g, n, case["gamma"])
    return _csr(keys, n, n, _values(g, keys.numel(), dt, 1, 255 if case["kind"] == "paths" else 100))


def _batch_sizes(case):
    c = case["count"]
    return [int(round(case["n_lo"] * (case["n_hi"] / case["n_lo"]) ** (b / max(1, c - 1)))) for b in range(c)]


def _inputs(case, seed):
    """The case's inputs, from the seed alone."""
    g, kind = _gen(seed), case["kind"]
    if kind in ("spgemm", "masked"):
        return {"A": _graph(case, g)}
    if kind == "batch":
        As = []
        for n in _batch_sizes(case):
            keys = _er_keys(g, n, case["d"])
            As.append(_csr(keys, n, n, _values(g, keys.numel(), case["dtype"])))
        return {"As": As}
    if kind == "paths":
        A = _graph(case, g)
        n, s = case["n"], case["nsrc"]
        has_out = torch.unique(A.col.long())
        src = has_out[torch.randperm(has_out.numel(), generator=g, device=DEV)[:s]]
        X0 = torch.full((n, src.numel()), NO_PATH, dtype=torch.int32, device=DEV)
        X0[src, torch.arange(src.numel(), device=DEV)] = 0
        return {"A": A, "X0": X0, "sources": src.cpu().numpy()}
    if kind == "apsp":
        n = case["n"]
        keys = torch.arange(n * n, device=DEV)
        keys = keys[keys // n != keys % n]
        if case["density"] < 1.0:
            keys = keys[torch.rand(keys.numel(), generator=g, device=DEV) < case["density"]]
        return {"A": _csr(keys, n, n, _values(g, keys.numel(), "i32", 1, n * n))}
    if kind == "gemm":
        dt = DTYPES[case["dtype"]]
        return {"A": torch.rand((case["m"], case["k"]), generator=g, device=DEV, dtype=dt),
                "B": torch.rand((case["k"], case["n"]), generator=g, device=DEV, dtype=dt)}
    if kind == "spmm":
        m, k, dt = case["m"], case["k"], case["dtype"]
        keys = torch.unique(torch.randint(0, m * k, (int(m * case["d"]),), generator=g, device=DEV))
        return {"A": _csr(keys, m, k, _values(g, keys.numel(), dt)),
                "X": _values(g, k * case["width"], dt).view(k, case["width"])}
    if kind == "fold":
        r, c = _rmat_pairs(g, case["n"], case["d"])
        return {"T": srtc.COO(r * case["n"] + c, _values(g, r.numel(), case["dtype"]), (case["n"],) * 2)}
    if kind == "jacobi":
        rowptr, col = _stencil(case["g"])
        n, dt = case["g"] ** 3, DTYPES[case["dtype"]]
        row = torch.repeat_interleave(torch.arange(n, device=DEV, dtype=torch.int32), torch.diff(rowptr))
        val = torch.where(row == col, 27.0, -1.0).to(dt)
        return {"A": srtc.CSR(rowptr, col, val, (n, n)), "b": torch.rand(n, generator=g, device=DEV, dtype=dt),
                "tol": case["rel"] * math.sqrt(n / 3.0)}
    i, j, k, dt = case["i"], case["j"], case["k"], case["dtype"]
    keys = torch.unique(torch.randint(0, i * j * k, (max(1, int(i * j * k * case["density"])),), generator=g, device=DEV))
    keys = keys[torch.randperm(keys.numel(), generator=g, device=DEV)]
    return {"T": srtc.COO(keys, _values(g, keys.numel(), dt), (i, j, k)),
            "M": _values(g, k * case["l"], dt).view(k, case["l"])}


_context = None


def _ctx():
    """One library context per process, as a program keeps."""
    global _context
    if _context is None:
        _context = srtc.Context(0)
    return _context


def prepare(case, seed):
    """Operands on the GPU, the caller's output buffers and the library's
    context."""
    st = _inputs(case, seed)
    st["kind"], st["ctx"] = case["kind"], _ctx()
    if case["kind"] == "paths":
        st["X"] = torch.empty_like(st["X0"])
    elif case["kind"] == "gemm":
        st["C"] = torch.empty((case["m"], case["n"]), dtype=st["A"].dtype, device=DEV)
    elif case["kind"] == "spmm":
        st["C"] = torch.empty((case["m"], case["width"]), dtype=st["X"].dtype, device=DEV)
        st["semiring"] = SEMIRING[case["dtype"]]
    elif case["kind"] == "jacobi":
        st["x"] = torch.empty_like(st["b"])
    elif case["kind"] == "tensor":
        st["C"] = torch.empty((case["i"], case["j"], case["l"]), dtype=st["M"].dtype, device=DEV)
    elif case["kind"] != "apsp":
        st["semiring"] = SEMIRING[case["dtype"]]
    return st


# ------------------------------------------------------------------ running --
def run(st):
    ctx, kind = st["ctx"], st["kind"]
    if kind == "spgemm":
        C = ctx.contract(st["semiring"], "ik", st["A"], "kj", st["A"], "ij")
        return {"rowptr": C.rowptr, "col": C.col, "val": C.val}
    if kind == "masked":
        C = ctx.contract_masked(st["semiring"], "ik", st["A"], "kj", st["A"], "ij", st["A"])
        return {"rowptr": C.rowptr, "col": C.col, "val": C.val}
    if kind == "batch":
        Cs = ctx.batch_contract(st["semiring"], st["As"], st["As"])
        return [(C.rowptr, C.col, C.val) for C in Cs]
    if kind == "paths":
        st["X"].copy_(st["X0"])
        steps = ctx.fixpoint("min_plus", st["A"], st["X"])
        levels, depth = ctx.bfs_levels(st["A"], st["sources"])
        return {"X": st["X"], "steps": steps, "levels": levels, "depth": depth}
    if kind == "apsp":
        D, H, rounds = ctx.apsp_tiskin(st["A"])
        return {"D": D, "H": H, "rounds": rounds}
    if kind == "gemm":
        return {"C": ctx.contract("plus_times", "ik", st["A"], "kj", st["B"], "ij", C=st["C"])}
    if kind == "spmm":
        return {"C": ctx.contract(st["semiring"], "ik", st["A"], "kj", st["X"], "ij", C=st["C"])}
    if kind == "fold":
        C = ctx.fold(st["semiring"], st["T"], "ij", "i", "j")
        return {"rowptr": C.rowptr, "col": C.col, "val": C.val}
    if kind == "jacobi":
        st["x"].zero_()
        steps, resid = ctx.jacobi(st["A"], st["b"], st["x"], tol=st["tol"])
        return {"x": st["x"], "steps": steps, "resid": resid}
    return {"C": ctx.contract("plus_times", "ijk", st["T"], "kl", st["M"], "ijl", C=st["C"])}


# --------------------------------------------------------------------- work --
def _rmat_sizes(n, d):
    """Expected (entries, products, outputs) of the square of an R-MAT graph:
    vertices with the same number of zero bits are alike, so rows are summed
    by class; an entry of probability p is present with 1 - exp(-edges p)."""
    s = max(1, (n - 1).bit_length())
    e = (1 << s) * d
    part = n / (1 << s)
    a, b, c, dd = ABCD
    lg = [math.lgamma(i + 1) for i in range(s + 1)]
    cols = [math.exp(lg[s] - lg[z] - lg[s - z]) for z in range(s + 1)]
    rows = []
    for z in range(s + 1):  # z zero bits in the row
        i, l = np.meshgrid(np.arange(z + 1), np.arange(s - z + 1), indexing="ij")
        cnt = np.exp(np.array([lg[z] - lg[u] - lg[z - u] for u in range(z + 1)])[:, None] +
                     np.array([lg[s - z] - lg[u] - lg[s - z - u] for u in range(s - z + 1)])[None, :])
        p = a ** i * b ** (z - i) * c ** (s - z - l) * dd ** l
        rows.append(float((cnt * -np.expm1(-e * p)).sum()))
    entries = sum(k * r for k, r in zip(cols, rows))
    products = sum(k * r * r for k, r in zip(cols, rows))
    m2 = (a * a + b * c, a * b + b * dd, c * a + dd * c, c * b + dd * dd)
    outputs = 0.0
    for x in range(s + 1):  # levels whose bit pairs are (0,0), (0,1), (1,0), (1,1)
        for y in range(s - x + 1):
            for z in range(s - x - y + 1):
                w = s - x - y - z
                cnt = math.exp(lg[s] - lg[x] - lg[y] - lg[z] - lg[w])
                mean = products * (m2[0] ** x * m2[1] ** y * m2[2] ** z * m2[3] ** w) / sum(m2) ** s
                outputs += cnt * -math.expm1(-mean)
    return entries * part ** 2, products * part ** 3, outputs * part ** 2


def _graph_sizes(case):
    graph = case.get("graph", "rmat")
    if graph == "stencil":
        g = case["g"]
        return (3 * g - 2) ** 3, (9 * g - 10) ** 3, (5 * g - 6) ** 3
    n = case["n"]
    if graph == "rmat":
        return _rmat_sizes(n, case["d"])
    if graph == "er":
        e, prod = n * case["d"], n * case["d"] ** 2
    else:
        mean = float((np.arange(1, n + 1) * _power_cdf(n, case["gamma"])).sum())
        e, prod = n * mean, n * mean * mean
    return e, prod, n * n * -math.expm1(-prod / (n * n))


def work(case):
    """Bytes: every input read once and every output written once (a matrix
    used twice counts once; expected sizes where the pattern is random).
    Flops: two per product that the result needs; a lower bound (none) where
    the iterations or the useful products depend on the data."""
    kind = case["kind"]
    es = SIZES[case.get("dtype", "i32")]
    if kind == "spgemm":
        e, prod, out = _graph_sizes(case)
        n = case["n"] if "n" in case else case["g"] ** 3
        return {"bytes": 16 * n + (4 + es) * (e + out), "flops": 2 * prod}
    if kind == "batch":
        by = fl = 0.0
        for n in _batch_sizes(case):
            e, prod, out = _graph_sizes({"graph": "er", "n": n, "d": case["d"]})
            by, fl = by + 16 * n + (4 + es) * (e + out), fl + 2 * prod
        return {"bytes": by, "flops": fl}
    if kind == "masked":
        e, _, _ = _graph_sizes(case)
        return {"bytes": 16 * case["n"] + 2 * (4 + es) * e, "flops": 0}
    if kind == "paths":
        e, _, _ = _graph_sizes(case)
        return {"bytes": 8 * case["n"] + 8 * e + 4 * 3 * case["n"] * case["nsrc"], "flops": 2 * e * case["nsrc"]}
    if kind == "apsp":
        n = case["n"]
        return {"bytes": 8 * n * n * case["density"] + 8 * n * n, "flops": 0}
    if kind == "gemm":
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": es * (m * k + k * n + m * n), "flops": 2 * m * n * k}
    if kind == "spmm":
        m, k, d, w = case["m"], case["k"], case["d"], case["width"]
        return {"bytes": 8 * m + (4 + es) * m * d + es * w * (m + k), "flops": 2 * m * d * w}
    if kind == "fold":
        e = case["n"] * case["d"]
        u, _, _ = _rmat_sizes(case["n"], case["d"])
        return {"bytes": (8 + es) * e + (4 + es) * u + 8 * case["n"], "flops": 0}
    if kind == "jacobi":
        g = case["g"]
        return {"bytes": (4 + es) * (3 * g - 2) ** 3 + (8 + 3 * es) * g ** 3, "flops": 2 * (3 * g - 2) ** 3}
    i, j, k, l = case["i"], case["j"], case["k"], case["l"]
    e = i * j * k * case["density"]
    return {"bytes": (8 + es) * e + es * (k * l + i * j * l), "flops": 2 * e * l}


# -------------------------------------------------------------------- exact --
def _products(A, lo, hi):
    """Keys i * n + j and fp64 values of the products of rows lo..hi-1 of A.A."""
    n = A.shape[1]
    a, b = int(A.rowptr[lo]), int(A.rowptr[hi])
    k = A.col[a:b].long()
    row = torch.repeat_interleave(torch.arange(lo, hi, device=DEV), torch.diff(A.rowptr[lo:hi + 1]))
    ln = A.rowptr[k + 1] - A.rowptr[k]
    at = torch.cumsum(ln, 0) - ln
    e = torch.repeat_interleave(torch.arange(k.numel(), device=DEV), ln)
    p = A.rowptr[k][e] + (torch.arange(e.numel(), device=DEV) - at[e])
    return row[e] * n + A.col[p].long(), A.val[a:b].double()[e] * A.val[p].double()


def _row_blocks(A, most=60_000_000):
    """Row ranges with at most `most` products each (at least one row)."""
    n = A.shape[0]
    ln = torch.diff(A.rowptr)
    per = torch.zeros(A.nnz + 1, dtype=torch.int64, device=DEV)
    per[1:] = torch.cumsum(ln[A.col.long()], 0)
    upto = per[A.rowptr].cpu().numpy()
    lo = 0
    while lo < n:
        hi = int(np.searchsorted(upto, upto[lo] + most, side="right")) - 1
        hi = min(n, max(lo + 1, hi))
        yield lo, hi
        lo = hi


def exact(case, seed):
    """Floating outputs in 64 bits with torch alone; None for integer ones
    and for results whose pattern is the whole question."""
    kind = case["kind"]
    if case.get("dtype") not in ("f64", "f32") or kind == "batch":
        return None
    st = _inputs(case, seed)
    if kind == "spgemm":
        vals = []
        for lo, hi in _row_blocks(st["A"]):
            key, v = _products(st["A"], lo, hi)
            key, order = torch.sort(key)
            _, seg = torch.unique_consecutive(key, return_inverse=True)
            if key.numel():
                out = torch.zeros(int(seg[-1]) + 1, dtype=torch.float64, device=DEV)
                vals.append(out.index_add_(0, seg, v[order]))
            del key, v, order, seg
        val = torch.cat(vals) if vals else torch.empty(0, dtype=torch.float64, device=DEV)
        return {"rowptr": None, "col": None, "val": val}
    if kind == "masked":
        A = st["A"]
        n = A.shape[1]
        row = torch.repeat_interleave(torch.arange(A.shape[0], device=DEV), torch.diff(A.rowptr))
        mask = row * n + A.col.long()
        out = torch.zeros(A.nnz, dtype=torch.float64, device=DEV)
        for lo, hi in _row_blocks(A):
            key, v = _products(A, lo, hi)
            at = torch.clamp(torch.searchsorted(mask, key), max=A.nnz - 1)
            hit = mask[at] == key
            out.index_add_(0, at[hit], v[hit])
        return {"rowptr": None, "col": None, "val": out[out != 0]}
    if kind == "gemm":
        return {"C": torch.matmul(st["A"].double(), st["B"].double())}
    if kind == "spmm":
        A, X = st["A"], st["X"]
        out = torch.empty((case["m"], case["width"]), dtype=torch.float64, device=DEV)
        step = max(1, int(4e8 / max(1.0, case["d"] * case["width"])))
        for lo in range(0, case["m"], step):
            hi = min(case["m"], lo + step)
            a, b = int(A.rowptr[lo]), int(A.rowptr[hi])
            row = torch.repeat_interleave(torch.arange(hi - lo, device=DEV), torch.diff(A.rowptr[lo:hi + 1]))
            part = torch.zeros((hi - lo, case["width"]), dtype=torch.float64, device=DEV)
            part.index_add_(0, row, A.val[a:b].double()[:, None] * X[A.col[a:b].long()].double())
            out[lo:hi] = part
        return {"C": out}
    if kind == "fold":
        key, order = torch.sort(st["T"].keys)
        _, seg = torch.unique_consecutive(key, return_inverse=True)
        out = torch.zeros(int(seg[-1]) + 1, dtype=torch.float64, device=DEV)
        out.index_add_(0, seg, st["T"].val[order].double())
        return {"rowptr": None, "col": None, "val": out}
    if kind == "jacobi":
        g, b = case["g"], st["b"].double().view(case["g"], case["g"], case["g"])
        tol = st["tol"]

        def around(x):
            """Sum over the 27 points around each one."""
            for d in range(3):
                y = x.clone()
                y.narrow(d, 1, g - 1).add_(x.narrow(d, 0, g - 1))
                y.narrow(d, 0, g - 1).add_(x.narrow(d, 1, g - 1))
                x = y
            return x

        x = torch.zeros_like(b)
        for it in range(10001):
            near = around(x) - x
            r = float((b - 27.0 * x + near).norm())
            if it > 0 and r <= tol:
                break
            x = (b + near) / 27.0
        return {"x": x.reshape(-1), "steps": None, "resid": None if case["dtype"] == "f32" else r}
    i, j, k, l = case["i"], case["j"], case["k"], case["l"]
    T, M = st["T"], st["M"].double()
    out = torch.zeros((i * j, l), dtype=torch.float64, device=DEV)
    for lo in range(0, T.keys.numel(), 1 << 21):
        ks = T.keys[lo:lo + (1 << 21)]
        out.index_add_(0, ks // k, T.val[lo:lo + (1 << 21)].double()[:, None] * M[ks % k])
    return {"C": out.view(i, j, l)}
