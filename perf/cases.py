"""The products that a user of this library has it compute, as cases to be timed.

Each case goes through the public entry points as a program calls them: a handle made and analysed once with the
automatic plan (CSR, and the packed sparse-times-dense product), or a call on the caller's arrays (COO, CSC, ELL).
The matrices are the library's own configurations and the shapes of its tests and benchmark: scattered uniform rows,
the 5-point and 27-point stencils, power-law rows, rows made of aligned runs of eight columns, and the random matrices
of density 0.01 with 2048 columns.  They are made on the GPU from the seed alone.

Columns of random rows are drawn with replacement and sorted inside the row (repeats add up, as the library allows), so
a matrix of another seed has other columns and, for power-law rows and random densities, other row lengths.
"""
import math

import torch

import paper_2603_07169_amd as s

DEVICE = "cuda"
LANES = 8  # columns in a run of the matrices made of aligned runs


def listed():
    return [
        # the smallest call in earnest use: 65536 entries, a few microseconds, where the launch is what counts
        {"name": "csr_uniform_4096_f32", "op": "csr", "kind": "uniform", "m": 4096, "n": 4096, "per_row": 16, "dtype": "f32", "beta": 0.0},
        # the benchmark's own shape of this product at its largest, bf16 storage
        {"name": "csr_density_32768_bf16", "op": "csr", "kind": "density", "m": 32768, "n": 2048, "density": 0.01, "dtype": "bf16", "beta": 0.0},
        # an iterative solver's product on a 2-D grid, with y kept (beta != 0)
        {"name": "csr_laplace2d_1024_f32", "op": "csr", "kind": "laplace2d", "grid": 1024, "dtype": "f32", "beta": 0.5},
        # a 3-D stencil in bf16 storage, a size that streams
        {"name": "csr_stencil27_128_bf16", "op": "csr", "kind": "stencil27", "grid": 128, "dtype": "bf16", "beta": 0.0},
        # a graph of moderate size with an odd number of rows: a few very long rows, x inside the caches
        {"name": "csr_powerlaw_333333_f32", "op": "csr", "kind": "powerlaw", "m": 333333, "dtype": "f32", "beta": 0.5},
        # a large graph: x fits no cache
        {"name": "csr_powerlaw_4M_f32", "op": "csr", "kind": "powerlaw", "m": 4000000, "dtype": "f32", "beta": 0.0},
        # a block-sparse matrix (rows of 16 runs of 8 columns) in bf16 storage
        {"name": "csr_blocks_1M_bf16", "op": "csr", "kind": "blocks", "m": 1000000, "runs": 16, "dtype": "bf16", "beta": 0.0},
        # sparse times dense at the benchmark's usual size: a layer with 1 % of its weights left, 4096 columns
        {"name": "spmm_65536x4096_f32", "op": "spmm", "kind": "density", "m": 65536, "n": 2048, "density": 0.01, "K": 4096, "dtype": "f32", "beta": 0.0},
        # the same in bf16 storage with ragged sizes and C kept
        {"name": "spmm_20011x1000_bf16", "op": "spmm", "kind": "density", "m": 20011, "n": 2048, "density": 0.01, "K": 1000, "dtype": "bf16", "beta": 0.5},
        # coordinate storage in row order, a size that streams
        {"name": "coo_stencil27_128_bf16", "op": "coo", "kind": "stencil27", "grid": 128, "dtype": "bf16", "beta": 0.0, "order": "rows"},
        # column storage, the benchmark's shape turned round
        {"name": "csc_density_2048x32768_f32", "op": "csc", "kind": "density", "m": 2048, "n": 32768, "density": 0.01, "dtype": "f32", "beta": 0.0},
        # padded rows, a size that streams
        {"name": "ell_stencil27_128_bf16", "op": "ell", "kind": "stencil27", "grid": 128, "dtype": "bf16", "beta": 0.0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: the products above over the sizes from their smallest to their largest, both storage types, with
    and without y (or C) kept."""
    op = rng.choice(["csr", "csr", "csr", "csr", "spmm", "spmm", "coo", "csc", "ell"])
    c = {"op": op, "dtype": rng.choice(["f32", "bf16"]), "beta": rng.choice([0.0, 0.0, 0.5])}
    if op == "csr":
        c["kind"] = rng.choice(["uniform", "density", "laplace2d", "stencil27", "powerlaw", "blocks"])
    elif op in ("spmm", "csc"):
        c["kind"] = "density"
    else:
        c["kind"] = rng.choice(["stencil27", "density"])
    k = c["kind"]
    if k == "uniform":
        c["m"] = c["n"] = _log_int(rng, 1000, 1000000)
        c["per_row"] = rng.randint(4, 32)
    elif k == "density":
        c["m"], c["n"] = _log_int(rng, 1024, 65536 if op == "spmm" else 32768), 2048
        if op in ("csc", "ell"):  # the benchmark's shapes of these layouts have few rows and many columns
            c["m"], c["n"] = 2048, c["m"]
        c["density"] = 0.01
        if op == "spmm":
            c["K"] = _log_int(rng, 64, 4096)
    elif k == "laplace2d":
        c["grid"] = _log_int(rng, 100, 1500)
    elif k == "stencil27":
        c["grid"] = _log_int(rng, 20, 128)
    elif k == "powerlaw":
        c["m"] = _log_int(rng, 20000, 4000000)
    else:
        c["m"] = LANES * _log_int(rng, 2000, 125000)
        c["runs"] = rng.randint(4, 16)
    if op == "coo":
        c["order"] = rng.choice(["rows", "rows", "any"])
    return c


# ---------------------------------------------------------------------------- inputs
def _generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    return g


def _pm1(g, *size):
    return torch.rand(*size, generator=g, device=DEVICE) * 2.0 - 1.0


def _sorted_columns(g, rows, n):
    """A column for every entry, uniform over [0, n), ascending inside each row; rows is ascending."""
    key = rows * n + torch.randint(0, n, (rows.numel(),), generator=g, device=DEVICE)
    key = torch.sort(key).values
    return key % n


def _stencil(shape, reach):
    """rows, columns of a stencil on a grid truncated at the faces; reach: offsets per axis, as tuples, in column order."""
    total = 1
    for d in shape:
        total *= d
    r = torch.arange(total, device=DEVICE)
    cols, ok = [], []
    for off in reach:
        inside = torch.ones(total, dtype=torch.bool, device=DEVICE)
        step, rest, stride = 0, r, 1
        for d, o in zip(shape[::-1], off[::-1]):
            at = rest % d + o
            inside &= (at >= 0) & (at < d)
            rest = torch.div(rest, d, rounding_mode="floor")
            step += o * stride
            stride *= d
        cols.append(r + step)
        ok.append(inside)
    ok = torch.stack(ok, 1)
    cols = torch.stack(cols, 1)
    rows = r[:, None].expand_as(cols)
    return total, rows[ok], cols[ok]


def _matrix(case, g):
    """m, n, rows (ascending), columns and float32 values of the case's matrix."""
    kind = case["kind"]
    if kind == "uniform":
        m, n = case["m"], case["n"]
        rows = torch.arange(m, device=DEVICE).repeat_interleave(case["per_row"])
        cols = _sorted_columns(g, rows, n)
        vals = _pm1(g, rows.numel())
    elif kind == "density":
        m, n = case["m"], case["n"]
        flat = torch.randint(0, m * n, (int(m * n * case["density"]),), generator=g, device=DEVICE)
        flat = torch.sort(flat).values
        rows, cols = torch.div(flat, n, rounding_mode="floor"), flat % n
        vals = _pm1(g, rows.numel())
    elif kind == "laplace2d":
        d = case["grid"]
        m, rows, cols = _stencil((d, d), [(-1, 0), (0, -1), (0, 0), (0, 1), (1, 0)])
        n = m
        vals = torch.where(rows == cols, 4.0, -1.0)
    elif kind == "stencil27":
        d = case["grid"]
        m, rows, cols = _stencil((d, d, d), [(a, b, c) for a in (-1, 0, 1) for b in (-1, 0, 1) for c in (-1, 0, 1)])
        n = m
        vals = torch.where(rows == cols, 26.0, _pm1(g, rows.numel()))
    elif kind == "powerlaw":  # row lengths 1 + floor(3.75 (u^(-2/3) - 1)), at most 200000: mean 8
        m = n = case["m"]
        u = 1.0 - torch.rand(m, generator=g, device=DEVICE, dtype=torch.float64)
        lens = (1.0 + torch.floor(3.75 * (u ** (-2.0 / 3.0) - 1.0))).clamp(max=min(200000, n)).to(torch.int64)
        rows = torch.arange(m, device=DEVICE).repeat_interleave(lens)
        cols = _sorted_columns(g, rows, n)
        vals = _pm1(g, rows.numel())
    else:  # blocks: every row holds `runs` aligned runs of eight consecutive columns
        m = n = case["m"]
        rows = torch.arange(m, device=DEVICE).repeat_interleave(case["runs"])
        first = _sorted_columns(g, rows, n // LANES) * LANES
        rows = rows.repeat_interleave(LANES)
        cols = (first[:, None] + torch.arange(LANES, device=DEVICE)).reshape(-1)
        vals = torch.randn(rows.numel(), generator=g, device=DEVICE)
    return m, n, rows, cols, vals


def _stored(case, t):
    return t.to(torch.bfloat16) if case["dtype"] == "bf16" else t.contiguous()


def _offsets(index, count):
    out = torch.zeros(count + 1, dtype=torch.int64, device=DEVICE)
    torch.cumsum(torch.bincount(index, minlength=count), 0, out=out[1:])
    return out.to(torch.int32)


def _inputs(case, seed):
    """The matrix, the dense operand and the old result, as the case stores them."""
    g = _generator(seed)
    m, n, rows, cols, vals = _matrix(case, g)
    if case["op"] == "spmm":
        x, y = _pm1(g, n, case["K"]), _pm1(g, m, case["K"])
    else:
        x, y = _pm1(g, n), _pm1(g, m)
    return m, n, rows, cols, _stored(case, vals), _stored(case, x), y


def prepare(case, seed):
    m, n, rows, cols, vals, x, y = _inputs(case, seed)
    op = case["op"]
    st = {"op": op, "m": m, "n": n, "nnz": vals.numel(), "x": x, "y": y, "alpha": 1.0, "beta": case["beta"],
          "code": s.SPMV_F32 if case["dtype"] == "f32" else s.SPMV_BF16, "stream": torch.cuda.current_stream().cuda_stream}
    if op in ("csr", "spmm"):
        st["A"] = s.CsrMatrix(m, n, _offsets(rows, m), cols.to(torch.int32), vals, st["code"], dict(prepare_spmm=1) if op == "spmm" else None)
    elif op == "coo":
        if case["order"] == "any":
            p = torch.randperm(vals.numel(), generator=_generator(seed + 1), device=DEVICE)
            rows, cols, vals = rows[p], cols[p], vals[p]
        st["row"], st["col"], st["vals"] = rows.to(torch.int32), cols.to(torch.int32), vals.contiguous()
    elif op == "csc":
        p = torch.sort(cols, stable=True).indices
        st["col_offsets"], st["row"], st["vals"] = _offsets(cols, n), rows[p].to(torch.int32), vals[p].contiguous()
    else:  # ell: rows padded to the longest, row-major, column -1 in a padding slot
        ptr = _offsets(rows, m).to(torch.int64)
        width = int((ptr[1:] - ptr[:-1]).max())
        slot = rows * width + torch.arange(rows.numel(), device=DEVICE) - ptr[rows]
        col_ids = torch.full((m * width,), -1, dtype=torch.int32, device=DEVICE)
        padded = torch.zeros(m * width, dtype=vals.dtype, device=DEVICE)
        col_ids[slot] = cols.to(torch.int32)
        padded[slot] = vals
        st["width"], st["col"], st["vals"] = width, col_ids, padded
    return st


def run(st):
    """One product y <- alpha*A*x + beta*y (C <- alpha*A*B + beta*C); returns the result vector (matrix)."""
    op, x, y = st["op"], st["x"], st["y"]
    if op == "csr":
        st["A"].run(x, y, st["alpha"], st["beta"], st["stream"])
    elif op == "spmm":
        st["A"].spmm(x, y, st["alpha"], st["beta"], st["stream"])
    elif op == "coo":
        s.check(s.spmv_coo_run(st["m"], st["n"], st["nnz"], st["row"].data_ptr(), st["col"].data_ptr(), st["vals"].data_ptr(), st["code"],
                               x.data_ptr(), y.data_ptr(), st["alpha"], st["beta"], st["stream"]), "spmv_coo_run")
    elif op == "csc":
        s.check(s.spmv_csc_run(st["m"], st["n"], st["nnz"], st["col_offsets"].data_ptr(), st["row"].data_ptr(), st["vals"].data_ptr(),
                               st["code"], x.data_ptr(), y.data_ptr(), st["alpha"], st["beta"], st["stream"]), "spmv_csc_run")
    else:
        s.check(s.spmv_ell_run(st["m"], st["n"], st["width"], st["col"].data_ptr(), st["vals"].data_ptr(), st["code"], x.data_ptr(),
                               y.data_ptr(), st["alpha"], st["beta"], st["stream"]), "spmv_ell_run")
    return y


# ---------------------------------------------------------------------------- what a case cannot do without
def _entries(case):
    """m, n and the number of stored entries (for power-law rows, whose lengths are random, their mean of 8 a row)."""
    kind = case["kind"]
    if kind == "uniform":
        return case["m"], case["n"], case["m"] * case["per_row"]
    if kind == "density":
        return case["m"], case["n"], int(case["m"] * case["n"] * case["density"])
    if kind == "laplace2d":
        d = case["grid"]
        return d * d, d * d, 5 * d * d - 4 * d
    if kind == "stencil27":
        d = case["grid"]
        return d ** 3, d ** 3, (3 * d - 2) ** 3
    if kind == "powerlaw":
        return case["m"], case["m"], 8 * case["m"]
    return case["m"], case["m"], case["m"] * case["runs"] * LANES


def work(case):
    """Every array of the storage layout read once and the result written once (read too where it is kept)."""
    m, n, nnz = _entries(case)
    e = 4 if case["dtype"] == "f32" else 2
    K = case.get("K", 1)
    op = case["op"]
    if op == "coo":
        index = 8 * nnz
    elif op == "csc":
        index = 4 * nnz + 4 * (n + 1)
    elif op == "ell":
        index = 4 * nnz
    else:
        index = 4 * nnz + 4 * (m + 1)
    return {"bytes": index + e * nnz + e * n * K + 4 * m * K * (2 if case["beta"] else 1), "flops": 2 * nnz * K}


def tolerance(case):
    """Products and sums are taken in binary32 on both storage types, so what another order of summation changes is a
    few units of 2^-24 (measured against 64 bits: 3e-8 to 3e-7)."""
    return {"rel": 1e-6, "max": 4e-5}


def exact(case, seed):
    """The same product in 64 bits."""
    m, n, rows, cols, vals, x, y = _inputs(case, seed)
    if case["op"] == "spmm":
        A = torch.zeros(m * n, dtype=torch.float64, device=DEVICE)
        A.index_add_(0, rows * n + cols, vals.double())
        out = torch.mm(A.view(m, n), x.double())
    else:
        out = torch.zeros(m, dtype=torch.float64, device=DEVICE)
        out.index_add_(0, rows, vals.double() * x.double()[cols])
    return out + case["beta"] * y.double() if case["beta"] else out
