"""GPU: the pipelined pattern kernel on grids whose blocks have one to sixteen runs of rows, at the sizes where its copies, sweeps
and rounds have remainders, in every shape it is compiled in; beyond its conditions the kernels that stand in for it.  What each case is
meant to reach is worked out from the matrix and asserted.  Integers, so that every path must give the oracle's result bit for
bit; a vals that is off its alignment takes the general path, an x that is off it the block kernel, and they are compared as well."""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_07169_amd as s
import workloads as w
from gpu_util import DeviceProblem, reference, to_dev

pytestmark = pytest.mark.gpu

SHEETS, RUNS, POSITIONS = "spmv_pattern_kernel", "spmv_pattern_block_kernel", "spmv_window_kernel"


def problem(name, dtype, m, n, rowptr, colidx, seed=5):
    rng = np.random.Generator(np.random.Philox(key=[np.uint64(seed), np.uint64(0)]))
    ints = lambda k: rng.integers(-4, 5, k).astype(np.float32)
    vals, x, y0 = ints(colidx.size), ints(n), ints(m)
    if dtype == "bf16":
        vals, x = w.f32_to_bf16_bits(vals), w.f32_to_bf16_bits(x)
    return w.CsrProblem(name, dtype, m, n, rowptr.astype(np.int32), colidx.astype(np.int32), vals, x, y0, 1.0, 2.0)


def grid(nx, lines, offsets, dtype, drop=None):
    """A stencil on `lines` lines of nx points: offsets are (lines, points) steps; rows in `drop` lose their entries."""
    m = nx * lines
    r = np.arange(m, dtype=np.int32)
    cols, ok = [], []
    kept = np.ones(m, bool)
    kept[[] if drop is None else drop] = False
    for dl, dx in offsets:
        line, at = r // nx + dl, r % nx + dx
        ok.append((line >= 0) & (line < lines) & (at >= 0) & (at < nx) & kept)
        cols.append(line * nx + at)
    ok, cols = np.stack(ok, 1), np.stack(cols, 1)
    return problem(f"grid_{nx}x{lines}", dtype, m, m, np.concatenate([[0], np.cumsum(ok.sum(1))]), cols[ok])


def spread(m, steps, dtype):
    """Row i has an entry at 8i + step for every step: as many x vectors as rows and far steps."""
    cols = 8 * np.arange(m, dtype=np.int32)[:, None] + np.asarray(sorted(steps), np.int32)
    return problem(f"spread_{m}_{len(steps)}", dtype, m, 8 * m + max(steps), len(steps) * np.arange(m + 1), cols.reshape(-1))


def reaches(p, block_nnz, rows_max, cus, beta):
    """(kernel, most runs of a block (0: some block has more than sixteen), lanes a row, x vectors a lane, blocks a workgroup at most) of the product, from the rules."""
    elem = 2 if p.dtype == "bf16" else 4
    blocks = oracle.row_blocks(p.rowptr, block_nnz, rows_max)
    nv, _, _, lidx = oracle.x_windows(p.rowptr, p.colidx, blocks, block_nnz, 16 // elem)
    few, many = (oracle.row_patterns(p.rowptr, blocks, lidx, block_nnz, max_runs=k) for k in (4, 16))
    other = RUNS if oracle.pattern_choice(p.nnz, few["covered"]) else POSITIONS
    runs, nb = many["n_runs"], blocks.size - 1
    if (runs == 0).any():
        return other, 0, 0, 0, 0
    if p.nnz // 32 >= p.m and nb <= (1 if elem == 4 else 2) * cus or 2 * 64 * np.count_nonzero(np.diff(p.rowptr) == 64) >= p.nnz:
        return other, int(runs.max()), 0, 0, 0
    sheet = 0
    for b in range(nb):
        at, lists = int(many["pat_ptr"][b]), set()
        for length in many["run_len"][b, :runs[b]].tolist():
            lists.add((length, many["pat"][at:at + length].tobytes()))
            at += length
        sheet = max(sheet, -(-rows_max // 16) * 16 + 16 * int(runs[b]) + sum((2 * k + 3) // 4 * 4 for k, _ in lists))
    sheet, x_cap, staged = -(-sheet // 16) * 16, max(int(nv.max()), 1), int(np.diff(p.rowptr[blocks]).max())
    buf = 16 * x_cap + -(-elem * (staged + 16) // 16) * 16 + sheet + (-(-4 * rows_max // 16) * 16 if beta else 0)
    if 2 * buf > 65536:
        return other, int(runs.max()), 0, 0, 0
    places = 160 * 1024 // (-(-2 * buf // 1280) * 1280)
    lanes = 2 if places * (2 if rows_max > 64 else 1) <= 10 and p.nnz // 16 >= p.m else 1
    wg = 128 * lanes
    per_lane = next(k for k in (1, 2, 4, 8) if x_cap <= k * wg)
    return SHEETS, int(runs.max()), lanes, per_lane, -(-nb // (min(places, 2048 // wg) * cus))


FIVE = [(-1, 0), (0, -1), (0, 0), (0, 1), (1, 0)]
BOX = lambda q: [(a, b) for a in range(-q, q + 1) for b in range(-q, q + 1)]
PLANES = lambda d: [(a + d * c, b) for c in (-1, 0, 1) for a in (-1, 0, 1) for b in (-1, 0, 1)]  # planes of d lines, not cut at their faces
FAR = [0, 3, 400000, 400003]                                                                    # two x vectors a row
FAR18 = [400000 * g + k for g in range(4) for k in range(4)] + [1600000, 1600001]                 # rows of 18 entries, five x vectors


# what makes the matrix, and its block_nnz and rows_max (None: the automatic ones); then (kernel, most runs of a block, lanes a row, x vectors a
# lane, least rounds: blocks of the busiest workgroup) for FP32 and for bf16
CASES = {
    "one_row": (lambda t: grid(1, 1, FIVE, t), None, (SHEETS, 1, 1, 1, 1)),                    # a window of less than one vector
    "three_rows": (lambda t: grid(3, 1, FIVE, t), None, (SHEETS, 3, 1, 1, 1)),
    "line_of_129": (lambda t: grid(129, 300, FIVE, t), None, (SHEETS, 4, 1, 1, 1)),
    "line_of_1027": (lambda t: grid(1027, 7, FIVE, t), None, (SHEETS, 4, 1, 1, 1)),            # the last x vector and the last value vector are incomplete
    "nine_of_77": (lambda t: grid(77, 201, BOX(1), t), None, (SHEETS, 4, 1, 1, 1)),
    "planes": (lambda t: grid(43, 200, PLANES(11), t), None, (SHEETS, 5, 1, 1, 1)),
    "line_of_64": (lambda t: grid(64, 64, BOX(2), t), None, (SHEETS, 6, 1, 1, 1)),
    "runs_12_rounds": (lambda t: grid(16, 45000, FIVE, t), (1024, 64), (SHEETS, 12, 1, 1, 3)),
    "runs_16": (lambda t: grid(14, 401, FIVE, t), None, (SHEETS, 16, 1, 1, 1)),
    "runs_16_rounds": (lambda t: grid(15, 47001, FIVE, t), (1024, 64), (SHEETS, 16, 1, 1, 3)),
    "runs_over_16": (lambda t: grid(9, 400, FIVE, t), None, (POSITIONS, 0, 0, 0, 0)),
    "long_rows": (lambda t: grid(301, 50, BOX(3), t), None, (SHEETS, 8, 1, 1, 1)),
    "long_rows_rounds": (lambda t: grid(301, 1100, BOX(3), t), None, (SHEETS, 8, 2, 1, 3)),
    "few_long_rows": (lambda t: grid(301, 10, BOX(3), t), None, (RUNS, 8, 0, 0, 0)),
    "rounds": (lambda t: grid(500, 1500, BOX(2), t), None, (SHEETS, 6, 2, 1, 3), (SHEETS, 6, 1, 1, 3)),
    "two_vectors_a_lane": (lambda t: spread(1 << 17, FAR, t), (2048, 128), (SHEETS, 1, 1, 2, 1)),
    "four_vectors_a_lane": (lambda t: spread(600_001, FAR, t), (2048, 256), (SHEETS, 1, 1, 4, 2)),
    "eight_vectors_a_lane": (lambda t: spread(1_000_001, FAR, t), (2048, 512), (SHEETS, 1, 1, 8, 3)),
    "two_lanes_two_vectors": (lambda t: spread(350_001, FAR18, t), (4096, 96), (SHEETS, 1, 2, 2, 3), (SHEETS, 1, 1, 4, 2)),
    "two_lanes_two_vectors_planes": (lambda t: grid(1000, 330, PLANES(40), t), (8192, 512), (RUNS, 4, 0, 0, 0), (SHEETS, 4, 2, 2, 1)),
    "two_lanes_four_vectors": (lambda t: spread(450_001, FAR18, t), (4096, 200), (SHEETS, 1, 2, 4, 3)),
    "blocks_of_1024_rows": (lambda t: grid(4000, 400, FIVE, t), (5120, 1024), (RUNS, 4, 0, 0, 0), (SHEETS, 4, 1, 4, 2)),  # FP32: two buffers pass 64 KB
}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", list(CASES))
def test_grids(case, dtype):
    make, shape, *want = CASES[case]
    p = make(dtype)
    params = dict(plan=s.SPMV_PLAN_WINDOWED)
    if shape:
        params.update(block_nnz=shape[0], rows_max=shape[1])
    run_both(p, params, want[-1 if dtype == "bf16" else 0])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_empty_rows_and_rows_off_the_pattern(dtype):
    p = grid(200, 90, FIVE, dtype, drop=np.r_[0, 1, 5, 300:700, 9000, 17999])
    run_both(p, dict(plan=s.SPMV_PLAN_WINDOWED))
    p.colidx = p.colidx.copy()
    for r in (40, 8000, 8003):               # one entry of these rows lies elsewhere
        p.colidx[p.rowptr[r]] += 1
    run_both(p, dict(plan=s.SPMV_PLAN_WINDOWED))


@pytest.mark.parametrize("rows_max", [1, 64, 127, 129, 1024])
def test_rows_of_a_block(rows_max):
    p = grid(160, 120, FIVE, "f32")
    run_both(p, dict(plan=s.SPMV_PLAN_WINDOWED, rows_max=rows_max, block_nnz=min(8192, 5 * rows_max)))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("kind", ["banded", "scattered"])
@pytest.mark.parametrize("length", [60, 64])
def test_rows_of_one_length(length, kind, dtype):
    """Rows of 64 entries meet on the same LDS banks: they go by the packed runs, or by their positions where nothing repeats; rows of
    60 go by their sheets, unless a block has more than sixteen different ones."""
    m, rng = 10_000, np.random.Generator(np.random.Philox(key=[np.uint64(length), np.uint64(1)]))
    if kind == "banded":
        steps = np.sort(rng.choice(128, length, replace=False))
    else:
        steps = np.sort(rng.random((m, 128)).argsort(1)[:, :length], 1)
    cols = np.arange(m)[:, None] + steps
    p = problem(f"rows_of_{length}_{kind}", dtype, m, m + 128, length * np.arange(m + 1), cols.reshape(-1))
    run_both(p, dict(plan=s.SPMV_PLAN_WINDOWED, block_nnz=1024, rows_max=64),
             (POSITIONS, 16 if length == 64 else 0, 0, 0, 0) if kind == "scattered" else (RUNS, 1, 0, 0, 0) if length == 64 else (SHEETS, 1, 1, 1, 1))


def test_planning_memory_is_given_back():
    """250000 blocks of one row: a handle keeps about 40 MB for them; what the sheets are planned in is not among it."""
    p = grid(500, 500, FIVE, "f32")
    d = DeviceProblem(p)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    A = d.matrix(dict(plan=s.SPMV_PLAN_WINDOWED, rows_max=1, block_nnz=5))
    kept = before - torch.cuda.mem_get_info()[0]
    assert A.info.num_row_blocks == p.m and s.spmv_csr_main_kernel_name(A.handle) == SHEETS
    want, _ = reference(p)
    assert np.array_equal(d.run(A).astype(np.float64), want)
    A.close()
    assert kept < 48 << 20, kept


def run_both(p, params, wanted=None):
    print("case", p.name, p.dtype, p.nnz, flush=True)
    aligned, general = DeviceProblem(p), DeviceProblem(p, offset_elems=1)
    off_x = DeviceProblem(p)
    off_x.x = to_dev(p.x, 1)
    A, G = aligned.matrix(params), general.matrix(params)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for beta in (0.0, 2.0):
        kernel, *shape = reaches(p, A.info.block_nnz, A.info.rows_max, cus, beta)
        if wanted:
            assert (kernel, *shape[:3]) == wanted[:4] and shape[3] >= wanted[4], (kernel, shape)
        want, _ = reference(p, 1.0, beta)
        for d, handle, name in ((aligned, A, kernel), (off_x, A, RUNS if A.info.lidx_patterned else POSITIONS),
                                (general, G, RUNS if G.info.lidx_patterned else POSITIONS)):
            assert s.spmv_csr_kernel_name(handle.handle, d.x.data_ptr(), beta) == name
            for _ in range(2):
                got = d.run(handle, 1.0, beta).astype(np.float64)
                assert np.array_equal(got, want), (p.name, name, beta, int(np.flatnonzero(got != want)[0]))
    A.close()
    G.close()
