"""The calls a user of this library makes, over the sizes they are made at.

A case names a matrix family with its sizes, the value type and the public
entry point: a plan's execute (default parameters or the selector's, rows
bound or searched), the one-call form, the allocation-free form, a batch, or
conjugate gradients.  Matrices are drawn on the GPU from the seed; the row
lengths of a random family are the quantiles of its distribution in a seeded
order, so a case's nonzero count does not depend on the seed.
"""
import functools
import math

import numpy as np
import torch

from paper_1504_06474_amd import sss

DTYPES = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}
VAL_BYTES = {"f64": 8, "f32": 4, "bf16": 2}
VEC_BYTES = {"f64": 8, "f32": 4, "bf16": 4}  # x and y: float for bf16 values


def listed():
    return [
        # one step of a small simulation: a 4,096-row matrix with empty rows,
        # default plan, where only launches and latency count
        {"name": "poisson_4k", "kind": "spmv", "family": "poisson", "size": 4096, "dtype": "f64",
         "via": "plan", "mode": "default", "bind": True},
        # a small web-like graph in single precision, rows of about 3 entries
        {"name": "weblike_30k_f32", "kind": "spmv", "family": "weblike", "size": 30011, "dtype": "f32",
         "via": "plan", "mode": "selector", "bind": True},
        # a program that keeps no plan: the one-call form on a 2D grid
        {"name": "onecall_grid_317", "kind": "spmv", "family": "stencil2d", "size": 317, "dtype": "f64",
         "via": "onecall", "mode": "default", "bind": False},
        # the benchmark's matrix class: 1M power-law rows of mean 20
        {"name": "powerlaw_1m", "kind": "spmv", "family": "powerlaw", "size": 1000000, "dtype": "f64",
         "via": "plan", "mode": "selector", "bind": True},
        # the same class stored in bfloat16, an odd number of rows
        {"name": "powerlaw_1m_bf16", "kind": "spmv", "family": "powerlaw", "size": 1000003, "dtype": "bf16",
         "via": "plan", "mode": "default", "bind": True},
        # a matrix whose x is far larger than any L2, single precision, from
        # a plan that serves any row_ptr of these sizes
        {"name": "zipf_4m_f32", "kind": "spmv", "family": "zipf", "size": 4000000, "dtype": "f32",
         "via": "plan", "mode": "default", "bind": False},
        # large regular matrices, which stream: a 27-point grid of 1.4 GB,
        # a finite-element band in single precision
        {"name": "grid3d_160", "kind": "spmv", "family": "stencil3d", "size": 160, "dtype": "f64",
         "via": "plan", "mode": "selector", "bind": True},
        {"name": "fem_778k_f32", "kind": "spmv", "family": "fem", "size": 777777, "dtype": "f32",
         "via": "plan", "mode": "selector", "bind": True},
        # large with short rows: the row structure is a good part of the work
        {"name": "grid2d_1414", "kind": "spmv", "family": "stencil2d", "size": 1414, "dtype": "f64",
         "via": "plan", "mode": "selector", "bind": True},
        # under capture or in a serving loop: the allocation-free form, a few
        # dense rows among short ones
        {"name": "noalloc_dense_rows", "kind": "spmv", "family": "dense", "size": 500009, "dtype": "f64",
         "via": "noalloc", "mode": "default", "bind": False},
        # many uneven matrices in one launch per stage, replayed as a graph
        {"name": "batch_256", "kind": "batch", "count": 256, "lo": 1000, "hi": 200000, "dtype": "f64", "graph": True},
        # the iterative use: 50 conjugate gradient steps on a 1M-row Laplacian
        {"name": "cg_1024", "kind": "cg", "size": 1024, "steps": 50},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# sizes of the families: rows, or a grid's side for the stencils
RANGES = {"poisson": (2000, 1000000), "weblike": (10000, 8000000), "powerlaw": (10000, 3000000),
          "zipf": (10000, 4000000), "dense": (5000, 1000000), "fem": (10000, 1500000),
          "stencil2d": (100, 2200), "stencil3d": (20, 160)}


def draw(rng):
    what = rng.random()
    if what < 0.1:
        return {"kind": "cg", "size": _log(rng, 64, 1024), "steps": rng.randint(10, 50)}
    if what < 0.25:
        lo = _log(rng, 500, 5000)
        return {"kind": "batch", "count": _log(rng, 8, 256), "lo": lo, "hi": _log(rng, 4 * lo, 200000),
                "dtype": rng.choice(["f64", "f32", "bf16"]), "graph": rng.random() < 0.5}
    family = rng.choice(sorted(RANGES))
    size = _log(rng, *RANGES[family])
    via = rng.choice(["plan", "plan", "plan", "onecall", "noalloc"])
    if via != "plan":
        return {"kind": "spmv", "family": family, "size": size, "dtype": "f64", "via": via, "mode": "default",
                "bind": False}
    return {"kind": "spmv", "family": family, "size": size, "dtype": rng.choice(["f64", "f64", "f32", "bf16"]),
            "via": via, "mode": rng.choice(["selector", "default"]), "bind": rng.random() < 0.75}


# ------------------------------------------------------------------ matrices

def _quantiles(cdf, m):
    """k such that cdf[k-1] <= u < cdf[k] at the m mid-quantiles u."""
    return np.minimum(np.searchsorted(cdf, (np.arange(m) + 0.5) / m, side="right"), len(cdf) - 1)


def _poisson(m, mean):
    k = np.arange(0, int(mean + 12 * math.sqrt(mean) + 12))
    logp = k * math.log(mean) - mean - np.array([math.lgamma(i + 1.0) for i in k])
    return _quantiles(np.cumsum(np.exp(logp)), m)


def _zipf(m, kmax, a, q):
    p = (np.arange(1, kmax + 1, dtype=np.float64) + q) ** -a
    return 1 + _quantiles(np.cumsum(p / p.sum()), m)


def _offset(kmax, a, mean):
    """q such that p(k) ~ (k + q)^-a on [1, kmax] has the given mean."""
    k = np.arange(1, kmax + 1, dtype=np.float64)
    lo, hi = 0.0, 4096.0
    for _ in range(40):
        mid = 0.5 * (lo + hi)
        p = (k + mid) ** -a
        if (k * p).sum() / p.sum() < mean:
            lo = mid
        else:
            hi = mid
    return 0.5 * (lo + hi)


@functools.lru_cache(maxsize=None)
def _offset_at(kmax, a, mean):
    return _offset(kmax, a, mean)


@functools.lru_cache(maxsize=8)
def _lengths(family, m):
    """The row lengths of a random family, before they are put in order."""
    if family == "poisson":  # mean 10, 5% of the rows empty
        out = np.minimum(_poisson(m, 10.0), m)
        out[:: 20] = 0
    elif family == "weblike":  # lognormal lengths of mean 3
        z = torch.special.ndtri((torch.arange(m, dtype=torch.float64) + 0.5) / m).numpy()
        out = np.minimum(np.rint(np.exp(math.log(3.0) - 0.5 + z)), m)
    elif family == "powerlaw":  # exponent 2 up to 2e5, mean 20, 3% empty
        kmax = min(m, 200000)
        out = _zipf(m, kmax, 2.0, _offset_at(kmax, 2.0, 20.0 / 0.97))
        out[np.arange(0, m, 33)] = 0
    elif family == "batch":  # exponent 2, mean 15
        kmax = min(m, 200000)
        out = _zipf(m, kmax, 2.0, _offset_at(2 ** (kmax.bit_length() - 1), 2.0, 15.0))
    elif family == "zipf":  # exponent 1.8, mean about 20
        out = _zipf(m, min(m, 42207), 1.8, 0.0)
    else:  # mean 5, and 8 dense rows of up to half the columns
        out = _poisson(m, 5.0)
        out[np.linspace(0, m - 1, 8).astype(np.int64)] = np.linspace(m // 100 + 1, m // 2, 8).astype(np.int64)
    return out.astype(np.int64)


def _nnz(case):
    family, s = case["family"], case["size"]
    if family == "stencil2d":
        return 5 * s * s - 4 * s
    if family == "stencil3d":
        return (3 * s - 2) ** 3
    if family == "fem":
        return s * min(50, s)
    return int(_lengths(family, s).sum())


def _rows(case):
    return case["size"] ** {"stencil2d": 2, "stencil3d": 3}.get(case["family"], 1)


def _random_rows(lengths, n, gen):
    """Sorted, distinct columns: entry j of a row of length L lies uniformly
    in the j-th of L equal parts of the columns."""
    dev = gen.device
    length = torch.from_numpy(lengths).to(dev)
    length = length[torch.randperm(length.numel(), generator=gen, device=dev)]
    rp = torch.zeros(length.numel() + 1, dtype=torch.int64, device=dev)
    torch.cumsum(length, 0, out=rp[1:])
    nnz = int(lengths.sum())
    each = torch.repeat_interleave(length, length, output_size=nnz)
    j = torch.arange(nnz, device=dev) - torch.repeat_interleave(rp[:-1], length, output_size=nnz)
    lo, hi = j * n // each, (j + 1) * n // each
    u = torch.rand(nnz, dtype=torch.float64, device=dev, generator=gen)
    col = lo + (u * (hi - lo)).to(torch.int64)
    return rp.to(torch.int32), torch.minimum(col, hi - 1).to(torch.int32)


def _grid(side, dims, dev):
    """A grid's neighbour columns and which of them exist, one row per point."""
    if dims == 2:
        steps = [(-1, 0), (0, -1), (0, 0), (0, 1), (1, 0)]
    else:
        steps = [(i, j, k) for i in (-1, 0, 1) for j in (-1, 0, 1) for k in (-1, 0, 1)]
    at = torch.arange(side ** dims, device=dev)
    where = [at // side ** (dims - 1 - d) % side for d in range(dims)]
    cols, there = [], []
    for step in steps:
        ok = torch.ones_like(at, dtype=torch.bool)
        c = at.clone()
        for d in range(dims):
            if step[d]:
                ok &= (where[d] + step[d] >= 0) & (where[d] + step[d] < side)
                c += step[d] * side ** (dims - 1 - d)
        cols.append(c.to(torch.int32))
        there.append(ok)
    return torch.stack(cols, 1), torch.stack(there, 1)


def _from_mask(cols, there):
    rp = torch.zeros(there.shape[0] + 1, dtype=torch.int64, device=cols.device)
    torch.cumsum(there.sum(1), 0, out=rp[1:])
    return rp.to(torch.int32), cols[there]


def _matrix(case, gen):
    """row_ptr, col and the column count of a case's matrix."""
    family, s, dev = case["family"], case["size"], gen.device
    if family in ("stencil2d", "stencil3d"):
        rp, col = _from_mask(*_grid(s, 2 if family == "stencil2d" else 3, dev))
        return rp, col, rp.numel() - 1
    if family == "fem":  # blocks of 10 rows share a 50-wide band near the diagonal
        w = min(50, s)
        base = torch.arange(-(-s // 10), device=dev) * 10 - w // 2
        base += torch.randint(-2 * w, 2 * w + 1, base.shape, generator=gen, device=dev)
        base = torch.repeat_interleave(base.clamp(0, s - w), 10)[:s]
        col = (base[:, None] + torch.arange(w, device=dev)).to(torch.int32).reshape(-1)
        return (torch.arange(s + 1, device=dev) * w).to(torch.int32), col, s
    rp, col = _random_rows(_lengths(family, s), s, gen)
    return rp, col, s


def _uniform(k, dtype, gen):
    return (torch.rand(k, dtype=torch.float64, device=gen.device, generator=gen) * 2 - 1).to(dtype)


def _generator(seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return gen


def _operands(case, rp, col, n, gen, y=None):
    val_dt = DTYPES[case["dtype"]]
    vec_dt = torch.float64 if case["dtype"] == "f64" else torch.float32
    if y is None:
        y = torch.zeros(rp.numel() - 1, dtype=vec_dt, device=gen.device)
    return {"rp": rp, "col": col, "n": n, "val": _uniform(col.numel(), val_dt, gen), "x": _uniform(n, vec_dt, gen),
            "y": y}


@functools.lru_cache(maxsize=4)
def _batch_sizes(count, lo, hi):
    """Row counts log-uniform in [lo, hi], as quantiles of that range."""
    return [int(round(lo * (hi / lo) ** ((i + 0.5) / count))) for i in range(count)]


def _batch_inputs(case, seed):
    gen = _generator(seed)
    sizes = _batch_sizes(case["count"], case["lo"], case["hi"])
    sizes = [sizes[i] for i in torch.randperm(len(sizes), generator=gen, device=gen.device).tolist()]
    y = torch.zeros(sum(sizes), dtype=torch.float64 if case["dtype"] == "f64" else torch.float32, device=gen.device)
    parts = torch.split(y, sizes)
    return [_operands(case, *_random_rows(_lengths("batch", m), m, gen), m, gen, part) for m, part in zip(sizes, parts)], y


def _spmv_inputs(case, seed):
    gen = _generator(seed)
    return _operands(case, *_matrix(case, gen), gen)


def _cg_inputs(case, seed):
    """The 5-point Laplacian and a random right-hand side."""
    gen = _generator(seed)
    cols, there = _grid(case["size"], 2, gen.device)
    rp, col = _from_mask(cols, there)
    val = torch.tensor([-1.0, -1.0, 4.0, -1.0, -1.0], dtype=torch.float64, device=gen.device).expand(cols.shape)[there]
    return rp, col, val, _uniform(rp.numel() - 1, torch.float64, gen)


# ------------------------------------------------------------------ the calls

def prepare(case, seed):
    if case["kind"] == "batch":
        mats, y = _batch_inputs(case, seed)
        plan = sss.BatchPlan([(a["rp"], a["col"], a["val"], a["x"], a["y"], a["n"]) for a in mats],
                             dtype=DTYPES[case["dtype"]])
        return {"kind": "batch", "plan": plan, "graph": case["graph"], "y": y}
    if case["kind"] == "cg":
        rp, col, val, b = _cg_inputs(case, seed)
        m = rp.numel() - 1
        plan = sss.Plan(m, m, col.numel(), mode=sss.MODE_SELECTOR, row_ptr=rp, bind_rows=True)
        work = torch.empty(sss.cg_workspace_size() // 8, dtype=torch.float64, device=b.device)
        x, r, p, q = (torch.zeros_like(b) for _ in range(4))
        return {"kind": "cg", "plan": plan, "rp": rp, "col": col, "val": val, "b": b, "x": x, "r": r, "p": p, "q": q,
                "work": work, "steps": case["steps"]}
    s = _spmv_inputs(case, seed)
    if case["via"] == "plan":
        mode = sss.MODE_SELECTOR if case["mode"] == "selector" else sss.MODE_FIXED
        s["plan"] = sss.Plan(s["rp"].numel() - 1, s["n"], s["col"].numel(), dtype=DTYPES[case["dtype"]], mode=mode,
                             row_ptr=s["rp"], bind_rows=case["bind"])
    s["kind"] = case["via"]
    return s


def run(s):
    kind = s["kind"]
    if kind == "plan":
        return s["plan"].execute(s["rp"], s["col"], s["val"], s["x"], s["y"])
    if kind == "onecall":
        return sss.csr_spmv(s["rp"], s["col"], s["val"], s["x"], s["y"])
    if kind == "noalloc":
        return sss.csr_spmv_noalloc(s["rp"], s["col"], s["val"], s["x"], s["y"])
    if kind == "batch":
        if s["graph"]:
            s["plan"].graph_launch()
        else:
            s["plan"].execute()
        return s["y"]
    s["x"].zero_()
    a = (s["plan"], s["rp"], s["col"], s["val"])
    sss.cg_start(*a, s["b"], s["x"], s["r"], s["p"], s["q"], s["work"])
    sss.cg_iterate(*a, s["x"], s["r"], s["p"], s["q"], s["work"], s["steps"])
    return {"x": s["x"], "r": s["r"], "p": s["p"], "scalars": s["work"][:3]}


def _bytes(m, n, nnz, dtype):
    return nnz * (4 + VAL_BYTES[dtype]) + 4 * (m + 1) + (m + n) * VEC_BYTES[dtype]


def work(case):
    """The matrix and x read once, y written once; a CG step also reads and
    writes its three vectors."""
    if case["kind"] == "batch":
        sizes = _batch_sizes(case["count"], case["lo"], case["hi"])
        nnz = [int(_lengths("batch", m).sum()) for m in sizes]
        return {"bytes": sum(_bytes(m, m, k, case["dtype"]) for m, k in zip(sizes, nnz)), "flops": 2 * sum(nnz)}
    if case["kind"] == "cg":
        m = case["size"] ** 2
        nnz = 5 * m - 4 * case["size"]
        return {"bytes": case["steps"] * (12 * nnz + 4 * (m + 1) + 6 * 8 * m),
                "flops": case["steps"] * (2 * nnz + 10 * m)}
    m, nnz = _rows(case), _nnz(case)
    return {"bytes": _bytes(m, m, nnz, case["dtype"]), "flops": 2 * nnz}


def _product(rp, col, val, x):
    products = val.double() * x.double()[col.to(torch.int64)]
    return torch.segment_reduce(products, "sum", lengths=(rp[1:] - rp[:-1]).to(torch.int64), unsafe=True, initial=0.0)


def exact(case, seed):
    if case["kind"] == "batch":
        return torch.cat([_product(a["rp"], a["col"], a["val"], a["x"]) for a in _batch_inputs(case, seed)[0]])
    if case["kind"] == "cg":
        rp, col, val, b = _cg_inputs(case, seed)
        x, r, p = torch.zeros_like(b), b.clone(), b.clone()
        rr = before = bb = torch.dot(b, b)
        for _ in range(case["steps"]):
            q = _product(rp, col, val, p)
            alpha = rr / torch.dot(p, q)
            x = x + alpha * p
            r = r - alpha * q
            before, rr = rr, torch.dot(r, r)
            p = r + (rr / before) * p
        return {"x": x, "r": r, "p": p, "scalars": torch.stack([rr, before, bb])}
    s = _spmv_inputs(case, seed)
    return _product(s["rp"], s["col"], s["val"], s["x"])
