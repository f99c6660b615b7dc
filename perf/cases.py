"""Timed cases of the CMRS library: the calls a user's program repeats.

A user converts CSR matrices to CMRS and back, multiplies (one right-hand
side with the default or a planned schedule, several right-hand sides, a
batch of matrices in one launch), and picks or trains the selector.  Each case
is one such call on one matrix (or batch) with every output buffer, plan and
workspace in place, as a solver loop or a serving loop keeps them.

Matrices are the families of the library's own workloads, made on the GPU
from the seed alone: 5-point and 27-point stencils, bands with 60 % fill,
Poisson row lengths with uniform columns, Zipf row lengths with 70 % of the
columns near the diagonal.  Values and x are N(0, 1).

`listed()` holds the cases, `draw()` gives one more of the same ranges,
`prepare()` / `run()` / `work()` / `exact()` make, run, price and compute one
in 64 bits.
"""
import math

import numpy as np
import torch

from paper_1203_2946_amd import cmrs, selector

DTYPES = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}
SIZE = {"f64": 8, "f32": 4, "bf16": 2}
ZIPF_A, ZIPF_MAX, ZIPF_NEAR, ZIPF_WINDOW = 2.0, 10_000, 0.7, 512


def listed():
    return [
        # The smallest call: a 64 x 64 grid's Laplacian, where a solver on a small system waits for launches.
        {"name": "spmv small grid", "op": "spmv", "family": "laplace", "rows": 4096, "mean": 5, "dtype": "f64",
         "height": 4, "variant": "auto"},
        # A 3-D finite-element-like matrix of two million rows at the selector's default class (height 8).
        {"name": "spmv stencil", "op": "spmv", "family": "stencil", "rows": 2_000_000, "mean": 27, "dtype": "f64",
         "height": 8, "variant": "auto"},
        # Uniform random columns, single precision, the paper's default height 4: bound by gathers.
        {"name": "spmv random columns", "op": "spmv", "family": "poisson", "rows": 1 << 20, "mean": 16,
         "dtype": "f32", "height": 4, "variant": "auto"},
        # The library's benchmark product: random columns, height 32, four concurrent column blocks.
        {"name": "colblock random columns", "op": "colblock", "family": "poisson", "rows": 1 << 20, "mean": 16,
         "dtype": "f64", "height": 32, "blocks": 4},
        # Skewed rows (up to 10^4 entries) with 16-bit values and the split schedule.
        {"name": "split skewed rows", "op": "split", "family": "zipf", "rows": 2_000_000, "mean": 0, "dtype": "bf16",
         "height": 32},
        # Conversion with the reorder, the first part of every pipeline, at the default height.
        {"name": "from_csr random columns", "op": "from_csr", "family": "poisson", "rows": 1 << 20, "mean": 16,
         "dtype": "f64", "height": 8, "sort": True},
        # The same for skewed rows, where a few strips hold a third of the entries.
        {"name": "from_csr skewed rows", "op": "from_csr", "family": "zipf", "rows": 2_000_000, "mean": 0,
         "dtype": "f32", "height": 16, "sort": True},
        # The way back, at the height of the benchmark step.
        {"name": "to_csr random columns", "op": "to_csr", "family": "poisson", "rows": 1 << 20, "mean": 16,
         "dtype": "f64", "height": 32},
        # A block solver's product: five right-hand sides, an odd row count.
        {"name": "spmm 5 columns", "op": "spmm", "family": "poisson", "rows": 131_071, "mean": 16, "dtype": "f64",
         "height": 4, "nrhs": 5},
        # An uneven batch (stencils and bands, 10 000 to 500 000 rows, 1 to 8 right-hand sides) in one launch.
        {"name": "batch of 32", "op": "batch", "family": "mixed", "rows": 500_000, "mean": 0, "dtype": "f64",
         "height": 8, "count": 32},
        # Choosing a class for a new matrix: its features, then the network.
        {"name": "select", "op": "select", "family": "band", "rows": 1_000_003, "mean": 20, "dtype": "f32",
         "height": 8},
        # One training step of the selector on its own data set: forward, loss gradient, backward.
        {"name": "train step", "op": "train", "family": "timings", "rows": 1500, "mean": 0, "dtype": "f32",
         "height": 8},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["spmv", "spmv", "colblock", "split", "from_csr", "from_csr", "to_csr", "spmm", "batch", "select",
                     "train"])
    if op == "train":
        return {"op": op, "family": "timings", "rows": _log_uniform(rng, 200, 2000), "mean": 0, "dtype": "f32",
                "height": 8}
    if op == "batch":
        return {"op": op, "family": "mixed", "rows": _log_uniform(rng, 100_000, 500_000), "mean": 0,
                "dtype": rng.choice(["f64", "f32"]), "height": rng.choice([2, 4, 8]), "count": rng.randint(4, 24)}
    dtype = rng.choice(["f64", "f64", "f32", "f32", "bf16"])
    if op == "colblock":
        # The gain of column blocks is for random columns and tall strips.
        return {"op": op, "family": "poisson", "rows": _log_uniform(rng, 200_000, 1_200_000),
                "mean": rng.randint(6, 24), "dtype": dtype, "height": rng.choice([8, 16, 32]),
                "blocks": rng.choice([4, 8])}
    if op == "split":
        return {"op": op, "family": "zipf", "rows": _log_uniform(rng, 100_000, 2_500_000), "mean": 0, "dtype": dtype,
                "height": rng.choice([8, 16, 32])}
    family = rng.choice(["laplace", "stencil", "band", "poisson", "zipf"])
    mean = {"laplace": 5, "stencil": 27, "band": rng.randint(8, 64), "poisson": rng.randint(2, 48), "zipf": 0}[family]
    rows = _log_uniform(rng, 2_000, 2_500_000)
    rows = min(rows, 40_000_000 // {"band": int(1.2 * mean) + 1, "zipf": 16}.get(family, mean))
    case = {"op": op, "family": family, "rows": rows, "mean": mean, "dtype": dtype,
            "height": rng.choice([1, 2, 4, 6, 8, 12, 16, 32])}
    if op == "spmv":
        case["variant"] = rng.choice(["auto", "auto", "lds_nt"])
    elif op == "from_csr":
        case["sort"] = rng.random() < 0.75
    elif op == "spmm":
        case["height"] = rng.choice([2, 4, 8])
        case["nrhs"] = rng.randint(1, 8)
        case["rows"] = min(rows, 8_000_000 // case["nrhs"] // max(mean, 6) * 4)
    return case


# ---------------------------------------------------------------- matrices
def _offsets_csr(n, offsets, keep):
    """CSR of the entries (i, i + offsets[k]) with keep[i, k]; offsets ascending."""
    dev = keep.device
    counts = keep.sum(1)
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device=dev)
    row_ptr[1:] = torch.cumsum(counts, 0)
    cols = torch.arange(n, device=dev, dtype=torch.int32)[:, None] + offsets.to(torch.int32)[None, :]
    return row_ptr.to(torch.int32), cols[keep]


def _distinct_csr(n, lengths, columns):
    """CSR of columns(r) per entry (r: its row), made distinct: each row's columns ascending plus their rank in the
    row, so `columns` stay below n - length."""
    dev = lengths.device
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device=dev)
    row_ptr[1:] = torch.cumsum(lengths, 0)
    r = torch.repeat_interleave(torch.arange(n, device=dev), lengths)
    key = torch.sort(r * n + columns(r)).values
    rank = torch.arange(r.numel(), device=dev) - row_ptr[r]
    return row_ptr.to(torch.int32), (key - r * n + rank).to(torch.int32)


def _grid_sides(family, rows):
    if family == "laplace":
        nx = max(2, round(math.sqrt(rows)))
        return nx, max(2, rows // nx), 1
    nx = max(2, round(rows ** (1 / 3)))
    return nx, nx, max(2, rows // (nx * nx))


def _size(family, rows):
    if family in ("laplace", "stencil"):
        nx, ny, nz = _grid_sides(family, rows)
        return nx * ny * nz
    return rows


def _pattern(family, rows, mean, g):
    """(row_ptr, col_ind, n) of a square matrix, columns ascending in every row."""
    dev = g.device
    n = _size(family, rows)
    i = torch.arange(n, device=dev)
    if family == "laplace":
        nx, ny, _ = _grid_sides(family, rows)
        x, y = i % nx, i // nx
        off = torch.tensor([-nx, -1, 0, 1, nx], device=dev)
        keep = torch.stack([y > 0, x > 0, torch.ones_like(x, dtype=torch.bool), x < nx - 1, y < ny - 1], 1)
        return (*_offsets_csr(n, off, keep), n)
    if family == "stencil":
        nx, ny, nz = _grid_sides(family, rows)
        x, y, z = i % nx, (i // nx) % ny, i // (nx * ny)
        off, keep = [], []
        for dz in (-1, 0, 1):
            for dy in (-1, 0, 1):
                for dx in (-1, 0, 1):
                    off.append(dx + dy * nx + dz * nx * ny)
                    keep.append((x + dx >= 0) & (x + dx < nx) & (y + dy >= 0) & (y + dy < ny) & (z + dz >= 0)
                                & (z + dz < nz))
        order = sorted(range(27), key=lambda k: off[k])
        keep = torch.stack([keep[k] for k in order], 1)
        off = torch.tensor([off[k] for k in order], device=dev)
        return (*_offsets_csr(n, off, keep), n)
    # Row lengths belong to the case, the columns to the seed: another seed has as many entries.
    shape = _generator(rows)
    if family == "band":
        off = torch.arange(-mean, mean + 1, device=dev)
        c = i.to(torch.int32)[:, None] + off.to(torch.int32)[None, :]
        inside = (c >= 0) & (c < n)
        k = (torch.rand(c.shape, generator=shape, device=dev) < 0.6).sum(1)
        k = torch.minimum(k, inside.sum(1)).clamp(min=1)
        u = torch.rand(c.shape, generator=g, dtype=torch.float64, device=dev).masked_fill_(~inside, 2.0)
        kth = torch.sort(u, dim=1).values.gather(1, k[:, None] - 1)
        return (*_offsets_csr(n, off, u <= kth), n)
    if family == "poisson":
        k = torch.poisson(torch.full((n,), float(mean), device=dev), generator=shape).clamp(1, n).to(torch.int64)

        def columns(r):
            return (torch.rand(r.numel(), generator=g, dtype=torch.float64, device=dev) * (n - k[r] + 1)).long()

        return (*_distinct_csr(n, k, columns), n)
    ks = torch.arange(1, ZIPF_MAX + 1, dtype=torch.float64, device=dev)
    cdf = torch.cumsum(ks ** -ZIPF_A, 0)
    u = torch.rand(n, generator=shape, dtype=torch.float64, device=dev)
    k = (torch.searchsorted(cdf / cdf[-1], u) + 1).clamp(max=min(ZIPF_MAX, n))

    def columns(r):
        near = torch.rand(r.numel(), generator=g, device=dev) < ZIPF_NEAR
        top = n - k[r]
        off = torch.randint(-ZIPF_WINDOW, ZIPF_WINDOW + 1, (r.numel(),), generator=g, device=dev)
        far = (torch.rand(r.numel(), generator=g, dtype=torch.float64, device=dev) * (top + 1)).long()
        return torch.where(near, torch.minimum((r - k[r] // 2 + off).clamp(min=0), top), far)

    return (*_distinct_csr(n, k, columns), n)


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _randn(shape, dtype, g):
    return torch.randn(shape, generator=g, dtype=torch.float32 if dtype == torch.bfloat16 else dtype,
                       device=g.device).to(dtype)


def _x_type(dtype):
    return torch.float64 if dtype == torch.float64 else torch.float32


def _csr(case, seed):
    """(row_ptr, col_ind, val, n, g) of the case's matrix."""
    g = _generator(seed)
    rp, ci, n = _pattern(case["family"], case["rows"], case["mean"], g)
    return rp, ci, _randn((ci.numel(),), DTYPES[case["dtype"]], g), n, g


def _batch_shapes(case):
    """(family, rows, mean, nrhs) of each matrix: rows spread over [10^4, rows] by their logarithm, stencils and
    bands in turn, right-hand sides 1..8 in turn; the sizes do not depend on the seed."""
    lo, hi, count = math.log(10_000), math.log(case["rows"]), case["count"]
    out = []
    for k in range(count):
        rows = int(round(math.exp(lo + (hi - lo) * (k + 0.5) / count))) | 1
        out.append(("stencil", rows, 27, 1 + (3 * k) % 8) if k % 2 == 0 else ("band", rows, 8 + (13 * k) % 57, 1 + (5 * k) % 8))
    return out


def _batch(case, seed):
    g = _generator(seed)
    dt = DTYPES[case["dtype"]]
    for family, rows, mean, nrhs in _batch_shapes(case):
        rp, ci, n = _pattern(family, rows, mean, g)
        val = _randn((ci.numel(),), dt, g)
        yield rp, ci, val, n, _randn((n, nrhs), _x_type(dt), g)


def _training(case, seed):
    """Rows of the committed timing set in a seeded order, targets, and freshly initialised parameters."""
    d = np.load(selector.DATA_PATH, allow_pickle=False)
    pick = np.random.default_rng(seed).permutation(d["features"].shape[0])[:case["rows"]]
    X = torch.from_numpy(d["features"][pick]).cuda()
    T = torch.from_numpy(selector.targets(d["times_ms"][pick])).cuda()
    return X, T, selector.init_params(int(seed) % (1 << 31))


# ---------------------------------------------------------------- the cases
def prepare(case, seed):
    op = case["op"]
    if op == "train":
        X, T, params = _training(case, seed)
        return {"op": op, "model": selector.Mlp(params), "X": X, "T": T}
    if op == "batch":
        mats, Xs, Ys = [], [], []
        for rp, ci, val, n, X in _batch(case, seed):
            mats.append(cmrs.from_csr(rp, ci, val, n, case["height"], sort=True))
            Xs.append(X)
            Ys.append(torch.empty_like(X))
        return {"op": op, "plan": cmrs.spmm_plan(mats, Xs, Ys), "Ys": Ys}
    rp, ci, val, n, g = _csr(case, seed)
    h = case["height"]
    if op == "select":
        return {"op": op, "csr": (rp, ci, n), "model": selector.load()}
    if op == "from_csr":
        nbytes = cmrs.from_csr_workspace_bytes(n, ci.numel(), h, case["sort"])
        out = cmrs.CmrsMatrix(n, n, h, cmrs.bits_for_height(h), case["sort"],
                              torch.empty(cmrs.num_strips(n, h) + 1, dtype=torch.int32, device=ci.device),
                              torch.empty_like(ci), torch.empty_like(val))
        return {"op": op, "csr": (rp, ci, val, n), "height": h, "sort": case["sort"], "out": out,
                "ws": torch.empty(max(nbytes, 1), dtype=torch.uint8, device=ci.device)}
    A = cmrs.from_csr(rp, ci, val, n, h, sort=True)
    if op == "to_csr":
        return {"op": op, "A": A, "out": (torch.empty_like(rp), torch.empty_like(ci), torch.empty_like(val))}
    xdt = _x_type(val.dtype)
    if op == "spmm":
        X = _randn((n, case["nrhs"]), xdt, g)
        return {"op": op, "A": A, "x": X, "y": torch.empty_like(X)}
    x = _randn((n,), xdt, g)
    s = {"op": op, "A": A, "x": x, "y": torch.empty_like(x)}
    if op == "spmv":
        s["variant"] = case["variant"]
    elif op == "colblock":
        s["plan"] = cmrs.colblock_plan(A, case["blocks"])
        s["ws"] = torch.empty(cmrs.spmv_colblock_workspace_bytes(A, case["blocks"], "concurrent"), dtype=torch.uint8,
                              device=x.device)
    else:
        s["plan"] = cmrs.split_plan(A)
    return s


def run(s):
    op = s["op"]
    if op == "spmv":
        return cmrs.spmv(s["A"], s["x"], out=s["y"], variant=s["variant"])
    if op == "colblock":
        return cmrs.spmv_colblock(s["A"], s["plan"], s["x"], out=s["y"], schedule="concurrent", workspace=s["ws"])
    if op == "split":
        return cmrs.spmv_split(s["A"], s["plan"], s["x"], out=s["y"])
    if op == "from_csr":
        rp, ci, val, n = s["csr"]
        M = cmrs.from_csr(rp, ci, val, n, s["height"], sort=s["sort"], workspace=s["ws"], out=s["out"])
        return M.strip_ptr, M.col_word, M.val
    if op == "to_csr":
        return cmrs.to_csr(s["A"], out=s["out"])
    if op == "spmm":
        return cmrs.spmm(s["A"], s["x"], out=s["y"])
    if op == "batch":
        cmrs.spmm_batched(s["plan"])
        return s["Ys"]
    if op == "select":
        f = selector.features(*s["csr"])
        return f, s["model"].predict(f.reshape(1, -1))
    return s["model"].grads(s["X"], s["T"])


# ---------------------------------------------------------------- what a pass cannot do without
def _nnz(family, rows, mean):
    """Entries of a matrix: exact for grids, the expected number for the random families."""
    n = _size(family, rows)
    if family == "laplace":
        nx, ny, _ = _grid_sides(family, rows)
        return 5 * nx * ny - 2 * nx - 2 * ny
    if family == "stencil":
        nx, ny, nz = _grid_sides(family, rows)
        return (3 * nx - 2) * (3 * ny - 2) * (3 * nz - 2)
    if family == "band":
        return int(n * 0.6 * (2 * mean + 1))
    if family == "poisson":
        return int(n * (mean + math.exp(-mean)))
    ks = np.arange(1, min(ZIPF_MAX, n) + 1, dtype=np.float64)
    return int(n * (ks ** (1 - ZIPF_A)).sum() / (np.arange(1, ZIPF_MAX + 1, dtype=np.float64) ** -ZIPF_A).sum())


def _product_work(nnz, n, h, sv, sx, nrhs):
    return {"bytes": (sv + 4) * nnz + 4 * (n // h + 2) + 2 * sx * nrhs * n, "flops": 2 * nnz * nrhs}


def work(case):
    op, h, sv = case["op"], case["height"], SIZE[case["dtype"]]
    sx = max(sv, 4)
    if op == "train":
        b = case["rows"]
        # Features, targets, parameters read; predictions and gradients written; three products per weight.
        return {"bytes": 4 * (b * (selector.N_FEATURES + 2 * selector.N_CLASSES) + 2 * selector.N_PARAMS),
                "flops": 6 * b * selector.N_PARAMS}
    if op == "batch":
        parts = [_product_work(_nnz(f, r, m), _size(f, r), h, sv, sx, k) for f, r, m, k in _batch_shapes(case)]
        return {key: sum(p[key] for p in parts) for key in ("bytes", "flops")}
    n = _size(case["family"], case["rows"])
    nnz = _nnz(case["family"], case["rows"], case["mean"])
    if op == "select":
        return {"bytes": 4 * (n + 1) + 4 * nnz + 4 * selector.N_PARAMS, "flops": 2 * selector.N_PARAMS}
    if op in ("from_csr", "to_csr"):
        return {"bytes": 4 * (n + 1) + 2 * (sv + 4) * nnz + 4 * (n // h + 2), "flops": 0}
    return _product_work(nnz, n, h, sv, sx, case.get("nrhs", 1))


# ---------------------------------------------------------------- the same in 64 bits
def _rows_of(rp, nnz):
    lengths = (rp[1:] - rp[:-1]).long()
    return torch.repeat_interleave(torch.arange(lengths.numel(), device=rp.device), lengths, output_size=nnz)


def _product(rp, ci, val, n, X):
    """A X in 64 bits, one column at a time."""
    r, c, v = _rows_of(rp, ci.numel()), ci.long(), val.double()
    cols = [torch.zeros(n, dtype=torch.float64, device=v.device).index_add_(0, r, v * x[c])
            for x in X.double().reshape(n, -1).unbind(1)]
    return torch.stack(cols, 1).reshape(X.shape)


def _features64(rp, ci, n):
    nnz = ci.numel()
    length = (rp[1:] - rp[:-1]).long().cpu().numpy()
    p = np.zeros(n, dtype=np.int64)
    p[length > 0] = np.frexp(length[length > 0].astype(np.float64))[1] - 1
    bins = np.where(length > 0, np.minimum(1 + 2 * p + (2 * length >= 3 * (1 << p)), 19), 0)
    dist = (ci.long() - _rows_of(rp, nnz)).abs().cpu().numpy()
    near = np.zeros(nnz, dtype=np.int64)
    near[dist > 0] = np.minimum(np.frexp(dist[dist > 0].astype(np.float64))[1], 15)
    tail = [math.log2(n) / 22, math.log2(nnz + 1) / 26, math.log2(nnz / n + 1) / 14,
            math.log2(int(length.max()) + 1) / 14]
    return torch.from_numpy(np.concatenate([np.bincount(bins, minlength=20) / n, np.bincount(near, minlength=16) / nnz,
                                            tail]))


def _layers(params):
    sizes = ((selector.N_FEATURES, selector.HIDDEN), (selector.HIDDEN, selector.HIDDEN),
             (selector.HIDDEN, selector.N_CLASSES))
    at = 0
    for i, o in sizes:
        yield params[at:at + i * o].reshape(i, o), params[at + i * o:at + i * o + o]
        at += i * o + o


def _network(X, params):
    (w1, b1), (w2, b2), (w3, b3) = _layers(params)
    h = torch.relu(torch.relu(X @ w1 + b1) @ w2 + b2)
    return h @ w3 + b3


def exact(case, seed):
    op = case["op"]
    if op == "train":
        X, T, params = _training(case, seed)
        params = params.double().requires_grad_()
        Y = _network(X.double(), params)
        ((Y - T.double()) ** 2).mean().backward()
        return Y.detach(), params.grad
    if op == "batch":
        return [_product(*part) for part in _batch(case, seed)]
    rp, ci, val, n, g = _csr(case, seed)
    if op == "select":
        f = _features64(rp, ci, n).cuda()
        return f, _network(f.reshape(1, -1), selector.load().params.double())
    if op == "from_csr":
        order = slice(None)
        h = case["height"]
        r = _rows_of(rp, ci.numel())
        if case["sort"]:
            order = torch.argsort(((r // h) * n + ci) * h + r % h, stable=True)
        word = (ci.long() << cmrs.bits_for_height(h) | r % h)[order]
        word = torch.where(word < 1 << 31, word, word - (1 << 32)).to(torch.int32)
        return torch.cat([rp[:-1:h], rp[-1:]]), word, val.double()[order]
    if op == "to_csr":
        return rp, ci, val.double()
    nrhs = case.get("nrhs")
    return _product(rp, ci, val, n, _randn((n, nrhs) if nrhs else (n,), _x_type(val.dtype), g))
