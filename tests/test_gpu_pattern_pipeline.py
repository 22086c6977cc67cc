"""GPU: the pipelined pattern kernel on grids whose blocks have one to sixteen and more runs of rows, at the sizes where its copies,
sweeps and rounds have remainders.  Integers, so that every path must give the oracle's result bit for bit; a vals that is off its
alignment takes the general path, and the two are compared as well."""
import numpy as np
import pytest
import torch

import paper_2603_07169_amd as s
import workloads as w
from gpu_util import DeviceProblem, reference

pytestmark = pytest.mark.gpu


def grid(nx, lines, offsets, dtype, drop=None, seed=5):
    """A stencil on `lines` lines of nx points: offsets are (lines, points) steps; rows in `drop` lose their entries."""
    m = nx * lines
    r = np.arange(m, dtype=np.int64)
    cols, ok = [], []
    for dl, dx in offsets:
        line, at = r // nx + dl, r % nx + dx
        ok.append((line >= 0) & (line < lines) & (at >= 0) & (at < nx) & ~np.isin(r, drop if drop is not None else []))
        cols.append(line * nx + at)
    ok, cols = np.stack(ok, 1), np.stack(cols, 1)
    rowptr = np.concatenate([[0], np.cumsum(ok.sum(1))]).astype(np.int32)
    colidx = cols[ok].astype(np.int32)
    rng = np.random.Generator(np.random.Philox(key=[np.uint64(seed), np.uint64(0)]))
    ints = lambda n: rng.integers(-4, 5, n).astype(np.float32)
    vals, x, y0 = ints(colidx.size), ints(m), ints(m)
    if dtype == "bf16":
        vals, x = w.f32_to_bf16_bits(vals), w.f32_to_bf16_bits(x)
    return w.CsrProblem(f"grid_{nx}x{lines}", dtype, m, m, rowptr, colidx, vals, x, y0, 1.0, 2.0)


FIVE = [(-1, 0), (0, -1), (0, 0), (0, 1), (1, 0)]
BOX = lambda q: [(a, b) for a in range(-q, q + 1) for b in range(-q, q + 1)]
PLANES = lambda d: [(a + d * c, b) for c in (-1, 0, 1) for a in (-1, 0, 1) for b in (-1, 0, 1)]  # planes of d lines, not cut at their faces

CASES = {
    "one_row": (1, 1, FIVE),                 # a window of less than one vector
    "three_rows": (3, 1, FIVE),
    "line_of_129": (129, 300, FIVE),
    "line_of_1027": (1027, 7, FIVE),         # the last x vector and the last value vector are incomplete
    "nine_of_77": (77, 201, BOX(1)),
    "runs_12": (43, 200, PLANES(11)),        # up to four lines a block
    "runs_over_16": (9, 400, FIVE),          # no sheet
    "line_of_64": (64, 64, BOX(2)),
    "long_rows": (301, 50, BOX(3)),          # 49 entries: two lanes a row
    "rounds": (500, 1500, BOX(2)),           # several blocks for every workgroup
}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", list(CASES))
def test_grids(case, dtype):
    nx, lines, offsets = CASES[case]
    p = grid(nx, lines, offsets, dtype)
    run_both(p, s.SPMV_PLAN_WINDOWED)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_empty_rows_and_rows_off_the_pattern(dtype):
    p = grid(200, 90, FIVE, dtype, drop=np.r_[0, 1, 5, 300:700, 9000, 17999])
    run_both(p, s.SPMV_PLAN_WINDOWED)
    p.colidx = p.colidx.copy()
    for r in (40, 8000, 8003):               # one entry of these rows lies elsewhere
        p.colidx[p.rowptr[r]] += 1
    run_both(p, s.SPMV_PLAN_WINDOWED)


@pytest.mark.parametrize("rows_max", [1, 64, 127, 129, 1024])
def test_rows_of_a_block(rows_max):
    p = grid(160, 120, FIVE, "f32")
    run_both(p, s.SPMV_PLAN_WINDOWED, dict(plan=s.SPMV_PLAN_WINDOWED, rows_max=rows_max, block_nnz=min(8192, 5 * rows_max)))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("kind", ["banded", "scattered"])
@pytest.mark.parametrize("length", [60, 64])
def test_rows_of_one_length(length, kind, dtype):
    """Rows of 64 entries meet on the same LDS banks: they go by the packed runs, or by their positions where nothing repeats; rows of
    60 go by their sheets, unless a block has more than sixteen different ones."""
    m, rng = 10_000, np.random.Generator(np.random.Philox(key=[np.uint64(length), np.uint64(1)]))
    n = m + 128
    first = np.arange(m)[:, None]
    if kind == "banded":
        cols = first + np.sort(rng.choice(128, length, replace=False))
    else:
        cols = first + np.sort(rng.random((m, 128)).argsort(1)[:, :length], 1)
    ints = lambda k: rng.integers(-4, 5, k).astype(np.float32)
    vals, x, y0 = ints(m * length), ints(n), ints(m)
    if dtype == "bf16":
        vals, x = w.f32_to_bf16_bits(vals), w.f32_to_bf16_bits(x)
    p = w.CsrProblem(f"rows_of_{length}_{kind}", dtype, m, n, (length * np.arange(m + 1)).astype(np.int32), cols.reshape(-1).astype(np.int32), vals, x, y0, 1.0, 2.0)
    kernel = "spmv_window_kernel" if kind == "scattered" else "spmv_pattern_block_kernel" if length == 64 else "spmv_pattern_kernel"
    run_both(p, s.SPMV_PLAN_WINDOWED, dict(plan=s.SPMV_PLAN_WINDOWED, block_nnz=1024, rows_max=64), kernel)


def test_planning_memory_is_given_back():
    """250000 blocks of one row: a handle keeps about 40 MB for them; the sheets' plan takes 69 MB more while it is made."""
    p = grid(500, 500, FIVE, "f32")
    d = DeviceProblem(p)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    A = d.matrix(dict(plan=s.SPMV_PLAN_WINDOWED, rows_max=1, block_nnz=5))
    kept = before - torch.cuda.mem_get_info()[0]
    assert A.info.num_row_blocks == p.m and s.spmv_csr_main_kernel_name(A.handle) == "spmv_pattern_kernel"
    want, _ = reference(p)
    assert np.array_equal(d.run(A).astype(np.float64), want)
    A.close()
    assert kept < 64 << 20, kept


def run_both(p, plan, params=None, kernel=None):
    print("case", p.name, p.dtype, p.nnz, flush=True)
    aligned, general = DeviceProblem(p), DeviceProblem(p, offset_elems=1)
    params = params or dict(plan=plan)
    A, G = aligned.matrix(params), general.matrix(params)
    assert kernel is None or s.spmv_csr_main_kernel_name(A.handle) == kernel
    for beta in (0.0, 2.0):
        want, _ = reference(p, 1.0, beta)
        got = aligned.run(A, 1.0, beta).astype(np.float64)
        assert np.array_equal(got, want), (p.name, beta, int(np.flatnonzero(got != want)[0]))
        assert np.array_equal(got, aligned.run(A, 1.0, beta))
        assert np.array_equal(got, general.run(G, 1.0, beta))
    A.close()
    G.close()
