"""GPU: the row-wise product with x gathered in column order (spmv_gather_kernel) - one chunk to a compute unit and four, chunks of
several rounds of words, cut rows, unaligned arrays, and the matrices that stay with the tile kernel - against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_07169_amd as s
import workloads as w
from gpu_util import DeviceProblem, assert_close, reference

pytestmark = pytest.mark.gpu

GATHER, TILE = "spmv_gather_kernel", "spmv_tile_kernel"


def problem(lens, n, dtype, seed=0, beta=0.5, width=None):
    """Integer-valued, so that every order of summation gives the same binary32 number: |sum| < 100000 * 32 < 2^24."""
    rng = np.random.default_rng(seed)
    lens = np.asarray(lens, dtype=np.int64)
    m = lens.size
    rowptr = np.concatenate(([0], np.cumsum(lens))).astype(np.int32)
    rows = np.repeat(np.arange(m, dtype=np.int64), lens)
    cols = rng.integers(0, n, rows.size) if width is None else np.clip(rows * n // m + rng.integers(0, width, rows.size), 0, n - 1)
    vals, x = rng.integers(-4, 5, rows.size).astype(np.float32), rng.integers(-8, 9, n).astype(np.float32)
    if dtype == "bf16":
        vals, x = ((a.view(np.uint32) >> 16).astype(np.uint16) for a in (vals, x))
    return w.CsrProblem(name="gather", dtype=dtype, m=m, n=n, rowptr=rowptr, colidx=cols.astype(np.int32), vals=vals, x=x,
                        alpha=1.0, beta=beta, y0=rng.integers(-8, 9, m).astype(np.float32))


def check(p, kernel, offset=0, params=None, runs=2):
    d = DeviceProblem(p, offset)
    A = d.matrix(params)
    assert s.spmv_csr_main_kernel_name(A.handle) == kernel
    y_ref, _ = reference(p)
    for _ in range(runs):  # the counters of cut rows are back at zero after a run
        assert np.array_equal(d.run(A), y_ref.astype(np.float32))
    return d, A


UNIFORM = {  # ADAPTIVE: rows x length, columns
    "rows_of_16": ([16] * 50000, 50000),                       # several lanes a row in binary32
    "odd": (np.random.default_rng(1).integers(0, 40, 50001), 9973),
    "least": {"f32": ([8] * 57344, 50000), "bf16": ([8] * 49152, 50000)},  # the fewest entries the rule takes
    "many_rows": ([3] * 131073, 50000),
    "long_rows": ([700] * 3000, 70000),                        # a wavefront a row
    "four_words_a_lane": ([16] * 220000, 100000),
    "four_chunks": ([16] * 300000, 100000),                    # binary32: four chunks to a compute unit; bf16: words in two rounds
    "banded": ([24] * 40000, 400000),
}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("name", list(UNIFORM))
def test_uncut_rows(name, dtype):
    lens, n = UNIFORM[name][dtype] if name == "least" else UNIFORM[name]
    p = problem(lens, n, dtype, beta=0.5, width=20000 if name == "banded" else None)
    d, A = check(p, GATHER, runs=1)
    assert A.info.plan == s.SPMV_PLAN_ADAPTIVE
    y_ref, _ = reference(p, 1.0, 0.0)  # an old y that is not to be read
    y = d.run(A, beta=0.0, y_init=torch.full((p.m,), float("nan"), device="cuda"))
    assert np.array_equal(y, y_ref.astype(np.float32))


def lengths_with(long_rows, short=60000, seed=3):
    lens = np.random.default_rng(seed).integers(0, 9, short)
    for at, length in long_rows:
        lens[at] = length
    return lens


CUT = {  # chunks that begin inside a row
    "first_and_last": lengths_with([(0, 3000), (59999, 5000)]),
    "neighbours": lengths_with([(i, 2500) for i in range(100, 130)]),      # both ends of a chunk inside rows
    "over_many_chunks": lengths_with([(7, 30000), (8, 513), (9, 40000)]),  # chunks without a row's end
    "all_long": [2900] * 150,
    "snapped": lengths_with([(i, 2048) for i in range(0, 60000, 800)] + [(77, 2049)]),     # the one row that chunks of up to 2048 steps cut
    "long_chunks": lengths_with([(i, 2048) for i in range(0, 60000, 400)] + [(77, 2049)]),  # beyond that, rows of more than 512 entries
    "next_to_empty_chunks": lengths_with([(i + j, 2048 if j == 1 else 2100) for i in range(0, 60, 6) for j in range(3)], short=9000),
    "empty_ends": np.concatenate(([0] * 5000, lengths_with([(100, 2500)]), [0] * 7000)),
}
UNCUT = {  # the same plan, no chunk begins inside a row
    "least": lengths_with([(5, 1100)], short=16200),                        # 65570 entries: the rule takes 65536
    "neighbours": lengths_with([(i, 1700) for i in range(100, 130)]),
    "over_empty_chunks": lengths_with([(i, 2048) for i in range(0, 60, 2)], short=9000),  # chunks of 512 steps: most are left empty
    "empty_ends": np.concatenate(([0] * 5000, lengths_with([(100, 2000)]), [0] * 7000)),
}
FULL = {  # storage, chunks to a compute unit, whether the pieces of cut rows are left to the second kernel
    "many_cuts_f32": ([100000] * 60, "f32", 4, True),
    "many_cuts_bf16": ([100000] * 110, "bf16", 4, True),
    "few_cuts": (lengths_with([(7, 30000), (99, 20000), (50000, 9000)], short=1200000), "f32", 4, False),
    "words_in_rounds": (lengths_with([(7, 30000), (99, 20000), (50000, 9000)], short=1200000), "bf16", 1, False),
}


def chunks_of(p, to_a_unit):
    """Steps of a chunk, and per chunk its first row, first entry and whether it begins inside a row: the oracle's merge path, with the cuts
    inside rows that a chunk does not cut moved back."""
    units = torch.cuda.get_device_properties(0).multi_processor_count * to_a_unit
    items = max(-(-(p.m + p.nnz) // units), 512)
    rows, entries = oracle.merge_path(p.rowptr, items)
    lens = np.append(np.diff(p.rowptr), 0)
    inside = p.rowptr[rows] < entries
    cut = inside & (lens[rows] > (2048 if items <= 2048 else 512))
    return items, rows, np.where(inside & ~cut, p.rowptr[rows], entries), cut


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("name", list(CUT))
def test_cut_rows(name, dtype):
    p = problem(CUT[name], 50000, dtype)
    items, _, entries, cut = chunks_of(p, 1)
    assert cut.any()
    if name == "neighbours":
        assert (cut[:-1] & cut[1:]).any()
    if name in ("snapped", "long_chunks"):
        longest = np.diff(p.rowptr)[oracle.merge_path(p.rowptr, items)[0][:-1][cut[:-1]]]
        assert set(longest) == {2049} if name == "snapped" else items > 2048
    if name == "next_to_empty_chunks":
        empty = np.diff(entries) == 0
        assert (cut[:-2] & empty[1:]).any() and (empty[:-1] & cut[2:]).any()  # an empty chunk behind a row's last piece, and one before its first
    _, A = check(p, GATHER)
    assert A.info.plan == s.SPMV_PLAN_MERGE


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("name", list(UNCUT))
def test_merge_plan_without_cut_rows(name, dtype):
    p = problem(UNCUT[name], 50000, dtype)
    _, _, entries, cut = chunks_of(p, 1)
    assert not cut.any()
    if name == "least":
        assert 1 << 16 <= p.nnz < (1 << 16) + 100
    if name == "over_empty_chunks":
        assert (np.diff(entries) == 0).sum() > 64
    _, A = check(p, GATHER)
    assert A.info.plan == s.SPMV_PLAN_MERGE


@pytest.mark.parametrize("name", list(FULL))
def test_cut_rows_of_full_chunks(name):
    lens, dtype, to_a_unit, second_kernel = FULL[name]
    p = problem(lens, 50000, dtype)
    for k in (1, 4):  # the fewest chunks whose values and x fit the LDS
        items, rows, entries, cut = chunks_of(p, k)
        slots = np.diff(entries).max()
        fits = items + 512 <= 32760 and (2 if dtype == "bf16" else 4) * 2 * slots + 8 * np.diff(rows).max() + 64 <= (160 - 8) * 1024 // min(k, 2)
        assert fits == (k == to_a_unit)
        if fits:
            break
    assert cut.any() and (12 * (cut.sum() - 600) > cut.size - 1) == second_kernel
    assert name != "words_in_rounds" or slots > 64 * 256  # 16 wavefronts, four words of a lane at a time
    _, A = check(p, GATHER)
    assert A.info.plan == s.SPMV_PLAN_MERGE


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("plan", ["adaptive", "merge"])
def test_unaligned_arrays(plan, dtype):
    lens = UNIFORM["odd"][0] if plan == "adaptive" else CUT["neighbours"]
    check(problem(lens, 9973, dtype), GATHER, offset=1)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_real_values(dtype):
    p = problem(CUT["neighbours"], 30000, dtype)
    rng = np.random.default_rng(5)
    vals, x = rng.standard_normal(p.nnz).astype(np.float32), rng.standard_normal(p.n).astype(np.float32)
    p.vals, p.x = (a if dtype == "f32" else (a.view(np.uint32) >> 16).astype(np.uint16) for a in (vals, x))
    d = DeviceProblem(p)
    A = d.matrix()
    y_ref, S_ref = reference(p)
    assert_close(p, d.run(A), y_ref, S_ref, p.alpha, p.beta)


def test_values_changed_in_place_and_non_finite_x():
    p = problem(UNIFORM["odd"][0], 9973, "f32", beta=0.0)
    d, A = check(p, GATHER)
    p.vals = -p.vals
    d.vals.neg_()
    assert np.array_equal(d.run(A), reference(p)[0].astype(np.float32))
    used = int(p.colidx[7])
    d.x[used] = float("inf")
    y = d.run(A)
    rows = np.unique(np.repeat(np.arange(p.m), np.diff(p.rowptr))[p.colidx == used])
    assert not np.isfinite(y[rows]).all() and np.isfinite(np.delete(y, rows)).all()


def test_matrices_of_the_tile_kernel():
    check(problem([8] * 57343, 50000, "f32"), TILE)                                      # too few entries
    check(problem([8] * 49151, 50000, "bf16"), TILE)
    check(problem([1000] * 2000, 12000, "bf16"), TILE)                                   # long rows, an x that a unit's cache holds
    check(problem([9000] * 900, 50000, "f32"), TILE)                                     # pieces of cut rows in nearly every chunk
    check(problem(lengths_with([(5, 1100)], short=16100), 50000, "f32"), TILE)            # too few entries, one row over the length of a block
    check(problem([40000] * 3, 100000, "f32"), TILE)                                     # rows over too many chunks
    check(problem([16] * 50000, 50000, "f32"), TILE, params=dict(plan=s.SPMV_PLAN_ADAPTIVE))
    check(problem(CUT["neighbours"], 50000, "f32"), TILE, params=dict(plan=s.SPMV_PLAN_MERGE))
    check(problem(CUT["neighbours"], 50000, "f32"), TILE, params=dict(prepare_spmm=1))   # a handle for products with matrices
    check(problem(CUT["neighbours"], 50000, "f32"), TILE, params=dict(items_per_chunk=512))
    check(problem([8] * 50000, 200_000_000, "bf16"), TILE)                               # neighbours too far apart for a word


def near(side, at, length, scattered):
    """A 2-D grid's five neighbours, and `scattered` columns anywhere in some rows: row lengths and columns."""
    m = side * side
    near_cols = np.arange(m)[:, None] + np.array([-side, -1, 0, 1, side])
    lens = np.full(m, 5)
    lens[at] = length
    cols = np.random.default_rng(7).integers(0, m, lens.sum())
    starts = np.concatenate(([0], np.cumsum(lens)[:-1]))
    for j in range(5):
        cols[starts + j] = np.clip(near_cols[:, j], 0, m - 1)
    if not scattered:
        cols = np.random.default_rng(8).permutation(m)[cols]
    return lens, cols, m


NEAR = {  # columns of neighbouring rows near each other, but for some rows; the same in no order
    "few_long_rows": lambda: near(800, [99, 300000], 4000, True),
    "block_of_scattered_rows": lambda: near(800, np.arange(999, 1063), 45, True),
    "long_rows_everywhere": lambda: near(600, np.arange(7, 360000, 300), 305, True),
    "short_call": lambda: near(440, np.arange(999, 1063), 45, True),
    "no_order": lambda: near(800, np.arange(999, 1063), 45, False),
    "no_order_cut": lambda: near(800, [99, 300000], 4000, False),
}


def lines_of(p, chunk_of_entry, chunks):
    """The 128-byte lines of x that the chunk with the most of them, all chunks, and all stretches of 1024 entries of a chunk touch."""
    line = p.colidx.astype(np.int64) // (64 if p.dtype == "bf16" else 32)
    per_chunk = np.bincount(np.unique(chunk_of_entry << 32 | line) >> 32, minlength=chunks)
    first = np.searchsorted(chunk_of_entry, np.arange(chunks))
    by_column = np.sort(chunk_of_entry << 32 | p.colidx) & 0xFFFFFFFF
    group = chunk_of_entry << 12 | (np.arange(p.nnz) - first[chunk_of_entry]) // 256
    starts = np.flatnonzero(np.append(True, group[1:] != group[:-1]))
    assert (np.maximum.reduceat(by_column, starts) - by_column[starts]).max() < (1 << 17) - 64  # nothing else speaks against the words
    stretch = chunk_of_entry << 12 | (np.arange(p.nnz) - first[chunk_of_entry]) // 1024
    return per_chunk.max(), per_chunk.sum(), np.unique(stretch << 32 | line).size


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("name", list(NEAR))
def test_the_lines_of_x_decide(name, dtype):
    """The kernel is the one that the rule gives for the lines as they are counted here."""
    lens, cols, n = NEAR[name]()
    p = problem(lens, n, dtype)
    p.colidx = cols.astype(np.int32)
    units = torch.cuda.get_device_properties(0).multi_processor_count
    _, _, entries, cut = chunks_of(p, 1)
    merge = name in ("few_long_rows", "no_order_cut")
    if not merge:  # no row is cut
        _, rows, _, _ = chunks_of(p, 1)
        entries = np.where(p.rowptr[rows] < entries, p.rowptr[rows], entries)
    chunk = np.repeat(np.arange(entries.size - 1), np.diff(entries))
    most, total, stretches = lines_of(p, chunk, entries.size - 1)
    saved = (stretches - total) / units - (most - total / (entries.size - 1))
    least = (-1250 if dtype == "bf16" else -2000) if merge else p.m / units * (11 if dtype == "bf16" else 4) / 16
    short = p.nnz + 4 * p.m <= 7680 * units
    assert short == (name == "short_call") and abs(saved - least) > 10  # the rule divides in whole numbers
    _, A = check(p, GATHER if short or saved >= least else TILE)
    assert A.info.plan == (s.SPMV_PLAN_MERGE if merge else s.SPMV_PLAN_ADAPTIVE)
    assert (saved >= least) == name.startswith("no_order")


GROUPS = {  # runs of eight a row, runs in x
    "blocks": ([8] * 70000, 5000),
    "odd": (np.random.default_rng(2).integers(0, 19, 60003), 4001),
    "long_rows": ([70] * 8000, 12500),
    "several_rounds": ([10] * 400000, 50000),
}


@pytest.mark.parametrize("name", list(GROUPS))
def test_groups_of_eight(name):
    runs, width = GROUPS[name]
    p = problem(runs, width, "bf16", seed=4)
    first = 8 * p.colidx.astype(np.int64)
    rng = np.random.default_rng(6)
    q = w.CsrProblem(name="groups", dtype="bf16", m=p.m, n=8 * width + 3, rowptr=8 * p.rowptr,
                     colidx=(first[:, None] + np.arange(8)).reshape(-1).astype(np.int32), vals=np.resize(p.vals, 8 * p.nnz),
                     x=(rng.integers(-8, 9, 8 * width + 3).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16), alpha=1.0, beta=0.5, y0=p.y0)
    d, A = check(q, "spmv_gather_group_kernel")
    assert A.info.plan == s.SPMV_PLAN_WINDOWED
    y_ref, _ = reference(q, 1.0, 0.0)
    assert np.array_equal(d.run(A, beta=0.0, y_init=torch.full((q.m,), float("nan"), device="cuda")), y_ref.astype(np.float32))
    moved = torch.empty(q.n + 1, dtype=torch.int16, device="cuda")[1:]  # an x that 16-byte reads do not fit: the windows
    moved.copy_(d.x)
    d.x = moved
    assert s.spmv_csr_kernel_name(A.handle, d.x.data_ptr(), q.beta) == "spmv_window_kernel"
    assert np.array_equal(d.run(A), reference(q)[0].astype(np.float32))
    if name == "blocks":
        check(q, "spmv_window_kernel", offset=1)                          # values that they do not fit
        check(q, "spmv_window_kernel", params=dict(prepare_spmm=1))


def consecutive(lens, first, n):
    """A bf16 problem whose rows' columns follow one another."""
    lens = np.asarray(lens, dtype=np.int64)
    rowptr = np.concatenate(([0], np.cumsum(lens)))
    cols = np.repeat(np.asarray(first), lens) + np.arange(rowptr[-1]) - np.repeat(rowptr[:-1], lens)
    assert rowptr[-1] >= 1 << 22 and cols.max() < n
    rng = np.random.default_rng(8)
    short = lambda size: (rng.integers(-8, 9, size).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)
    return w.CsrProblem(name="consecutive", dtype="bf16", m=lens.size, n=n, rowptr=rowptr.astype(np.int32), colidx=cols.astype(np.int32),
                        vals=short(cols.size), x=short(n), alpha=1.0, beta=0.5, y0=rng.integers(-8, 9, lens.size).astype(np.float32))


def ends(lens):
    return np.concatenate(([0], np.cumsum(lens)[:-1]))


NOT_GROUPS = {  # grouped positions, but rows that begin or end inside a group, or groups at columns that are no multiple of eight
    "diagonal": lambda: consecutive([1] * ((1 << 22) + 5), np.arange((1 << 22) + 5), (1 << 22) + 5),
    "rows_of_4": lambda: consecutive([4] * (1 << 20), 4 * np.arange(1 << 20), 1 << 22),
    "rows_of_12": lambda: consecutive([12] * 400000, 12 * np.arange(400000), 4800000),
    "rows_of_4_and_12": lambda: consecutive([4, 12] * 300000, ends([4, 12] * 300000), 4800000),
    "short_last_row": lambda: consecutive([8] * 599999 + [5], 8 * np.arange(600000), 4800000),
    "band": lambda: consecutive([16] * 300000, np.arange(300000), 300015),
}


@pytest.mark.parametrize("name", list(NOT_GROUPS))
def test_grouped_positions_that_are_no_groups_stay_with_the_windows(name):
    p = NOT_GROUPS[name]()
    _, A = check(p, "spmv_window_kernel")
    assert A.info.plan == s.SPMV_PLAN_WINDOWED and A.info.lidx_grouped == 1


def test_graph_replays_and_streams():
    p = problem(UNIFORM["odd"][0], 9973, "f32")
    d, A = check(p, GATHER)
    y_ref = reference(p)[0].astype(np.float32)
    y = torch.zeros(p.m, device="cuda")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        A.run(d.x, y, 1.0, p.beta, torch.cuda.current_stream().cuda_stream)
    for _ in range(3):
        y.copy_(d.y0)
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy(), y_ref)
        assert np.array_equal(d.run(A), y_ref)
    streams, ys = [torch.cuda.Stream() for _ in range(2)], [d.y0.clone() for _ in range(2)]
    torch.cuda.synchronize()
    for st, out in zip(streams, ys):  # an adaptive handle keeps no scratch: its runs may overlap
        A.run(d.x, out, 1.0, p.beta, st.cuda_stream)
    torch.cuda.synchronize()
    assert all(np.array_equal(out.cpu().numpy(), y_ref) for out in ys)
