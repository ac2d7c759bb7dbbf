"""Performance cases: the work a program that uses this framework has it do.

Every case goes through the package's public entry points (conversion, staging
of x, SpMV, the plain-CSR kernels, batches, the request server) on the matrix
families the benchmark and the tests use: 2D 5-point Laplacians, weighted
27-point stencils, rows of power-law length and of uniform random length with
random columns, and shifted Laplacians for the server's solves.  ``listed()``
names twelve of them, ``draw()`` gives others of the same ranges.

All inputs are made on the GPU from a seed.  Values are FP32 numbers held as
FP64, so that storing them as BF16 or FP16 is one rounding.
"""
import math

import numpy as np
import torch

import paper_1203_5737_amd as ac
from paper_1203_5737_amd import serve

DTYPES = {"f64": ac.F64, "f32": ac.F32, "bf16": ac.BF16, "f16": ac.F16}
VALUE_BYTES = {"f64": 8, "f32": 4, "bf16": 2, "f16": 2}
MAX_ROW = 10_000          # longest power-law row
UNIFORM_ROW = (5, 50)     # nonzeros per row of the uniform random matrices


def listed():
    return [
        # the smallest call: one product with a 64 x 64 Laplacian, where the
        # host path and the launch are all there is
        dict(name="spmv-laplace2d-f64", do="spmv", matrix="laplace2d", n=64 * 64, dtype="f64",
             block_dim=64, desired=1, staged="no"),
        # irregular rows (circuit and optimisation matrices), the benchmark's
        # headline: 10^6 rows, a few of 10^4 nonzeros, random columns
        dict(name="spmv-powerlaw-f64", do="spmv", matrix="powerlaw", n=1_000_000, dtype="f64",
             block_dim=64, desired=1, staged="no"),
        # the same family at an odd middle size in FP32
        dict(name="spmv-powerlaw-f32", do="spmv", matrix="powerlaw", n=333_667, dtype="f32",
             block_dim=128, desired=1, staged="no"),
        # regular rows (finite differences, structural matrices) at the
        # benchmark's size, as converted without further steps
        dict(name="spmv-stencil27-f64", do="spmv", matrix="stencil27", n=128 ** 3, dtype="f64",
             block_dim=128, desired=27, staged="no"),
        # the same matrix as an iterative solver in FP32 keeps it: x staged
        dict(name="spmv-stencil27-f32-staged", do="spmv", matrix="stencil27", n=128 ** 3,
             dtype="f32", block_dim=128, desired=27, staged="lds"),
        # 2-byte values on a grid whose side is no multiple of anything
        dict(name="spmv-stencil27-bf16-staged", do="spmv", matrix="stencil27", n=101 ** 3,
             dtype="bf16", block_dim=128, desired=27, staged="lds"),
        # many small and middle matrices in one launch
        dict(name="batch-f32", do="batch", members=48, n_lo=1_000, n_hi=200_000, dtype="f32"),
        # a program that has its matrix in CSR and uses it a few times only:
        # the plain-CSR kernel with the rows binned by length once
        dict(name="csr-binned-powerlaw-f64", do="csr", matrix="powerlaw", n=1_000_000,
             dtype="f64", lanes=-1),
        # a matrix assembled on the GPU is converted there
        dict(name="convert-powerlaw-f64", do="convert", matrix="powerlaw", n=1_000_000,
             dtype="f64", block_dim=64, desired=1, grouping="device"),
        # a matrix read by the host (its row offsets are there) is converted
        dict(name="convert-stencil27-f32", do="convert", matrix="stencil27", n=100 ** 3,
             dtype="f32", block_dim=128, desired=27, grouping="host"),
        # x of a converted banded matrix is staged and the first product of a
        # solve made
        dict(name="stage-stencil27-f32", do="stage", matrix="stencil27", n=100 ** 3,
             dtype="f32", block_dim=128, desired=27),
        # a burst of requests to a server with resident matrices: products
        # and solves to a residual of 1e-10, all in flight together
        dict(name="serve-burst", do="serve", matrices=4, n_lo=10_000, n_hi=300_000, spmv=8,
             cg=8),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    do = rng.choice(["spmv"] * 6 + ["csr", "convert", "convert", "stage", "batch", "serve"])
    dtype = rng.choice(list(DTYPES))
    if do == "batch":
        return dict(do=do, members=rng.randint(2, 48), n_lo=_log(rng, 1_000, 5_000),
                    n_hi=_log(rng, 20_000, 200_000), dtype=dtype)
    if do == "serve":
        return dict(do=do, matrices=rng.randint(1, 4), n_lo=_log(rng, 5_000, 20_000),
                    n_hi=_log(rng, 40_000, 300_000), spmv=rng.randint(1, 8), cg=rng.randint(1, 8))
    banded = do == "stage" or rng.random() < 0.5
    if banded:
        matrix = rng.choice(["stencil27", "stencil27", "laplace2d"])
        big = 100 if do in ("stage", "convert") else 128
        n = _log(rng, 8, big) ** 3 if matrix == "stencil27" else _log(rng, 40, 1_000) ** 2
        desired = 27 if matrix == "stencil27" else 5
    else:
        matrix = rng.choice(["powerlaw", "powerlaw", "uniform"])
        n = _log(rng, 1_000, 1_000_000 if matrix == "powerlaw" else 500_000)
        desired = 1 if matrix == "powerlaw" else rng.choice([1, 8, 27])
    if do == "csr":
        return dict(do=do, matrix=matrix, n=n, dtype=dtype, lanes=rng.choice([-1, 0]))
    block_dim = rng.choice([64, 128, 128, 256])
    c = dict(do=do, matrix=matrix, n=n, dtype=dtype, block_dim=block_dim, desired=desired)
    if do == "spmv":
        c["staged"] = rng.choice(["no", "lds", "lds", "gather"]) if banded else "no"
    elif do == "convert":
        c["grouping"] = rng.choice(["device", "host"])
    return c


# ---- matrices ---------------------------------------------------------------

def _generator(seed, *key):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1_000_003 + sum((k + 1) * 7919 ** i for i, k in enumerate(key)))
                  % (1 << 62))
    return g


def _uniform(n, lo, hi, g):
    """U[lo, hi): FP32 numbers held as FP64."""
    return (torch.rand(n, generator=g, device="cuda") * (hi - lo) + lo).double()


def _csr(row_len, col, val, n_cols):
    row_ptr = torch.zeros(row_len.numel() + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(row_len, 0, out=row_ptr[1:])
    row_ptr = row_ptr.to(torch.int32)
    return ac.DeviceCsr(row_len.numel(), n_cols, row_ptr.cpu().numpy(), row_ptr,
                        col.to(torch.int32).contiguous(), val.contiguous())


def _random_columns(row_len, n_cols, g):
    """Ascending distinct random columns per row: entry j of a row of L lies
    in the j-th of L equal parts of the columns."""
    first = torch.cumsum(row_len, 0) - row_len
    row = torch.repeat_interleave(torch.arange(row_len.numel(), device="cuda"), row_len)
    j = torch.arange(row.numel(), device="cuda") - first[row]
    L = row_len[row]
    lo, hi = j * n_cols // L, (j + 1) * n_cols // L
    u = torch.rand(row.numel(), generator=g, device="cuda", dtype=torch.float64)
    return lo + torch.clamp((u * (hi - lo)).long(), max=hi - lo - 1)


def _zipf_cdf(longest):
    """P(L <= k), k = 1..longest, for L = min(Zipf(2), longest)."""
    p = 1.0 / np.arange(1, longest + 1, dtype=np.float64) ** 2 / (math.pi ** 2 / 6)
    c = np.cumsum(p)
    c[-1] = 1.0
    return c


def _powerlaw(n, g):
    # the row lengths follow from n: every seed gives arrays of the same sizes
    cdf = torch.from_numpy(_zipf_cdf(min(MAX_ROW, n))).cuda()
    u = torch.rand(n, generator=_generator(0, n), device="cuda", dtype=torch.float64)
    L = torch.clamp(torch.searchsorted(cdf, u) + 1, max=cdf.numel())
    col = _random_columns(L, n, g)
    return _csr(L, col, _uniform(col.numel(), -1.0, 1.0, g), n)


def _uniform_rows(n, g):
    L = torch.randint(UNIFORM_ROW[0], UNIFORM_ROW[1] + 1, (n,), generator=_generator(0, n),
                      device="cuda")
    L = torch.clamp(L, max=n)
    col = _random_columns(L, n, g)
    return _csr(L, col, _uniform(col.numel(), -1.0, 1.0, g), n)


def _grid(shape, offsets, value):
    """Rows of a stencil on a grid, neighbours outside the grid left out;
    value(offset, rows) gives one column of values."""
    n = math.prod(shape)
    strides = [math.prod(shape[d + 1:]) for d in range(len(shape))]
    offsets = sorted(offsets, key=lambda o: sum(a * b for a, b in zip(o, strides)))
    rows = torch.arange(n, device="cuda")
    coords = [(rows // strides[d]) % shape[d] for d in range(len(shape))]
    there = torch.empty((n, len(offsets)), dtype=torch.bool, device="cuda")
    val = torch.empty((n, len(offsets)), dtype=torch.float64, device="cuda")
    shift = torch.empty(len(offsets), dtype=torch.int64, device="cuda")
    for k, o in enumerate(offsets):
        m = torch.ones(n, dtype=torch.bool, device="cuda")
        for d, step in enumerate(o):
            if step:
                m &= (coords[d] + step >= 0) & (coords[d] + step < shape[d])
        there[:, k] = m
        shift[k] = sum(a * b for a, b in zip(o, strides))
        val[:, k] = value(o, rows)
    col = (rows[:, None] + shift[None, :])[there]
    return _csr(there.sum(1), col, val[there], n)


def _star(dim):
    return [tuple(0 for _ in range(dim))] + [tuple(s if e == d else 0 for e in range(dim))
                                             for d in range(dim) for s in (-1, 1)]


def _side(n, dim):
    return max(2, int(round(n ** (1.0 / dim))))


def _stencil27(n, g):
    """Couplings -w, w ~ U[0.5, 1.5), and a diagonal that dominates them."""
    s = _side(n, 3)
    box = [(a, b, c) for a in (-1, 0, 1) for b in (-1, 0, 1) for c in (-1, 0, 1)]
    return _grid((s, s, s), box, lambda o, r: _uniform(r.numel(), 27.0, 40.0, g) if o == (0, 0, 0)
                 else -_uniform(r.numel(), 0.5, 1.5, g))


def _laplace2d(n, g):
    """5-point stencil with varying coefficients."""
    s = _side(n, 2)
    return _grid((s, s), _star(2), lambda o, r: _uniform(r.numel(), 4.0, 5.0, g) if o == (0, 0)
                 else -_uniform(r.numel(), 0.5, 1.0, g))


def _shifted_laplacian(dim, n, g):
    """2*dim on the diagonal plus U[0, 1), -1 beside it: symmetric positive
    definite, as a solve needs it."""
    s = _side(n, dim)
    zero = tuple(0 for _ in range(dim))
    return _grid((s,) * dim, _star(dim),
                 lambda o, r: _uniform(r.numel(), 0.0, 1.0, g) + 2.0 * dim if o == zero
                 else torch.full((r.numel(),), -1.0, dtype=torch.float64, device="cuda"))


MATRICES = {"powerlaw": _powerlaw, "uniform": _uniform_rows, "stencil27": _stencil27,
            "laplace2d": _laplace2d}


def _rows(matrix, n):
    """(rows, mean nonzeros per row) of a matrix family at n."""
    if matrix == "powerlaw":
        cdf = _zipf_cdf(min(MAX_ROW, n))
        return n, float(np.sum(1.0 - cdf) + 1.0)
    if matrix == "uniform":
        return n, sum(UNIFORM_ROW) / 2.0
    if matrix == "stencil27":
        s = _side(n, 3)
        return s ** 3, (3 - 2 / s) ** 3
    s = _side(n, 2)
    return s * s, 5 - 4 / s


def _member(case, k):
    """(matrix family, rows) of member k of a batch: the sizes spread over
    their logarithm, uniform and power-law rows in turn."""
    f = (k + 0.5) / case["members"]
    n = int(round(case["n_lo"] * (case["n_hi"] / case["n_lo"]) ** f))
    return ("uniform" if k % 2 == 0 else "powerlaw"), n


def _resident(case, k):
    """(dimension, rows) of matrix k of a server."""
    f = (k + 0.5) / case["matrices"]
    n = int(round(case["n_lo"] * (case["n_hi"] / case["n_lo"]) ** f))
    return 2 + k % 2, n


def _stored(csr, dtype):
    """The values as a case stores them."""
    return csr.val.to(ac.storage_dtype(DTYPES[dtype]))


def _vector(n, dtype, g):
    return _uniform(n, -1.0, 1.0, g).to(ac.vector_dtype(DTYPES[dtype]))


# ---- the cases --------------------------------------------------------------

def _inputs(case, seed):
    g = _generator(seed)
    A = MATRICES[case["matrix"]](case["n"], g)
    return A, _vector(A.n_cols, case["dtype"], g)


def _batch_inputs(case, seed):
    got = []
    for k in range(case["members"]):
        g = _generator(seed, k + 1)
        family, n = _member(case, k)
        A = MATRICES[family](n, g)
        got.append((A, _vector(A.n_cols, case["dtype"], g)))
    return got


def _serve_inputs(case, seed):
    mats = []
    for k in range(case["matrices"]):
        dim, n = _resident(case, k)
        mats.append(_shifted_laplacian(dim, n, _generator(seed, k + 1)))
    g = _generator(seed, 0)
    asks = []
    for i in range(case["spmv"] + case["cg"]):
        kind = "spmv" if i % 2 == 0 and i // 2 < case["spmv"] or i // 2 >= case["cg"] else "cg"
        if sum(a[0] == kind for a in asks) >= case[kind]:
            kind = "cg" if kind == "spmv" else "spmv"
        m = i % case["matrices"]
        v = _uniform(mats[m].n_cols, -1.0, 1.0, g)
        asks.append((kind, m, v.float() if kind == "spmv" else v))
    return mats, asks


def prepare(case, seed):
    do = case["do"]
    if do == "serve":
        mats, asks = _serve_inputs(case, seed)
        srv = serve.Server(budget_bytes=2 << 30)
        tickets = [srv.admit(k, A.row_ptr_host, A.col.cpu().numpy(), A.val.cpu().numpy(),
                             A.n_cols) for k, A in enumerate(mats)]
        for t in tickets:
            srv.wait(t)
            srv.release(t)
        return dict(do=do, srv=srv, rows=[A.n_rows for A in mats],
                    asks=[(kind, m, v.cpu().numpy()) for kind, m, v in asks])
    if do == "batch":
        dt = DTYPES[case["dtype"]]
        mats, xs, ys = [], [], []
        for A, x in _batch_inputs(case, seed):
            r = ac.autotune_member(A.row_ptr_host, dt)
            mats.append(ac.convert(A, r["block_dim"], r["desired_chunk_size"], dt,
                                   fmt=r["format"]))
            xs.append(x)
            ys.append(torch.empty(A.n_rows, dtype=x.dtype, device="cuda"))
        return dict(do=do, batch=ac.Batch(mats, xs, ys), ys=ys)
    A, x = _inputs(case, seed)
    dt = DTYPES[case["dtype"]]
    if do == "csr":
        return dict(do=do, A=A, x=x, dtype=dt, values=_stored(A, case["dtype"]),
                    lanes=case["lanes"], bins=ac.csr_bins(A) if case["lanes"] < 0 else None)
    if do == "convert":
        return dict(do=do, A=A, block_dim=case["block_dim"], desired=case["desired"], dtype=dt,
                    device=case["grouping"] == "device")
    M = ac.convert(A, case["block_dim"], case["desired"], dt)
    if do == "stage":
        return dict(do=do, M=M, x=x)
    if case["staged"] != "no":
        M = ac.stage(M, gap=0, lds=case["staged"] == "lds")
    return dict(do=do, M=M, x=x)


def _bits(values):
    """Stored values as whole numbers: a conversion is exact."""
    return values.view({8: torch.int64, 4: torch.int32, 2: torch.int16}[values.element_size()])


def run(state):
    do = state["do"]
    if do == "spmv":
        return ac.spmv(state["M"], state["x"])
    if do == "csr":
        if state["bins"] is None:
            return ac.csr_spmv(state["A"], state["x"], values=state["values"],
                               dtype=state["dtype"], lanes_per_row=state["lanes"])
        return ac.csr_spmv_binned(state["A"], state["x"], state["bins"],
                                  values=state["values"], dtype=state["dtype"])
    if do == "batch":
        state["batch"].launch()
        return state["ys"]
    if do == "convert":
        M = ac.convert(state["A"], state["block_dim"], state["desired"], state["dtype"],
                       device_grouping=state["device"])
        return {"groups": M.groups, "mapping": M.threads_mapping, "columns": M.columns,
                "values": _bits(M.values), "heavy": M.heavy_groups}
    if do == "stage":
        M = ac.stage(state["M"], gap=0)
        return {"tile_ptr": M.tile_ptr, "tile_start": M.tile_start, "tile_len": M.tile_len,
                "local": M.local, "y": ac.spmv(M, state["x"])}
    srv = state["srv"]
    asked = [srv.spmv(m, v, state["rows"][m]) if kind == "spmv" else srv.cg(m, v)
             for kind, m, v in state["asks"]]
    for ticket, _ in asked:
        if srv.wait(ticket)["status"] != 0:
            raise RuntimeError("a request failed")
        srv.release(ticket)
    return [out for _, out in asked]


def _spmv_work(rows, nnz, dtype):
    sx = 8 if dtype == "f64" else 4
    return {"bytes": nnz * (VALUE_BYTES[dtype] + 4) + rows * (4 + 2 * sx), "flops": 2 * nnz}


def work(case):
    do = case["do"]
    if do == "serve":
        w = {"bytes": 0, "flops": 0}
        sizes = [_resident(case, k) for k in range(case["matrices"])]
        for i in range(case["spmv"] + case["cg"]):
            dim, n = sizes[i % len(sizes)]
            one = _spmv_work(n, n * (2 * dim + 1), "f64")
            w = {k: w[k] + one[k] for k in w}
        return w
    if do == "batch":
        w = {"bytes": 0, "flops": 0}
        for k in range(case["members"]):
            rows, mean = _rows(*_member(case, k))
            one = _spmv_work(rows, rows * mean, case["dtype"])
            w = {k: w[k] + one[k] for k in w}
        return w
    rows, mean = _rows(case["matrix"], case["n"])
    nnz = rows * mean
    if do == "convert":
        return {"bytes": nnz * (12 + 4 + VALUE_BYTES[case["dtype"]]) + 8 * rows, "flops": 0}
    w = _spmv_work(rows, nnz, case["dtype"])
    if do == "stage":
        w["bytes"] += nnz * 2
    return w


# ---- the same in 64 bits ----------------------------------------------------

def _row_of(A):
    return torch.repeat_interleave(torch.arange(A.n_rows, device="cuda"),
                                   (A.row_ptr[1:] - A.row_ptr[:-1]).long())


def _product(A, val, x, row=None):
    y = torch.zeros(A.n_rows, dtype=torch.float64, device="cuda")
    return y.index_add_(0, _row_of(A) if row is None else row, val.double() * x.double()[A.col.long()])


def _solve(A, b):
    """Conjugate gradients to a residual of 1e-14."""
    row = _row_of(A)
    x = torch.zeros_like(b)
    r, p = b.clone(), b.clone()
    rr = torch.dot(r, r)
    stop = 1e-28 * float(rr)
    for _ in range(2000):
        if float(rr) <= stop:
            break
        q = _product(A, A.val, p, row)
        alpha = rr / torch.dot(p, q)
        x += alpha * p
        r -= alpha * q
        new = torch.dot(r, r)
        p = r + (new / rr) * p
        rr = new
    return x


def exact(case, seed):
    do = case["do"]
    if do == "convert":
        return None                      # whole numbers: compared as they are
    if do == "serve":
        mats, asks = _serve_inputs(case, seed)
        return [_product(mats[m], mats[m].val.float(), v) if kind == "spmv" else _solve(mats[m], v)
                for kind, m, v in asks]
    if do == "batch":
        return [_product(A, _stored(A, case["dtype"]), x) for A, x in _batch_inputs(case, seed)]
    A, x = _inputs(case, seed)
    y = _product(A, _stored(A, case["dtype"]), x)
    if do == "stage":
        return {"tile_ptr": None, "tile_start": None, "tile_len": None, "local": None, "y": y}
    return y
