"""GPU: rows that chunk boundaries cut into pieces (merge-path and two-pass plans, and the product without a handle).  Inputs
are small integers, so every order of summation gives the same numbers: the results equal the oracle's bit for bit, run after
run (the arrival counters wrap by themselves)."""
import time

import numpy as np
import pytest
import torch

import oracle
import paper_2603_07169_amd as s
import workloads as w
from gpu_util import DTYPE_CODE, DeviceProblem

pytestmark = pytest.mark.gpu

SNAP = 256        # merge-path cuts inside rows of at most this many entries (or items_per_chunk - 1) are moved to the row's first entry
LENGTHS = {
    "around_the_snap": [255, 256, 257, 3, 0, 512, 513] * 40,
    "one_row_over_many_chunks": [5] * 700 + [60000] + [1] * 300,
    "long_rows_side_by_side": [3000, 2500, 0, 0, 4097, 2048, 2047, 1, 8193, 512],
    "ends_on_a_cut": [2047, 2047, 4095, 1, 2046, 10000],     # row ends on steps that are multiples of 2048
    "starts_and_ends_long": [9000] + [2] * 5000 + [9000],
}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("name", LENGTHS)
def test_cut_rows_bit_for_bit_run_after_run(name, dtype):
    lens = LENGTHS[name]
    p = w.exact_integer(lens, 70000, seed=11, dtype=dtype, alpha=2.0, beta=-1.0)
    y_ref, _ = oracle.spmv_problem(p)
    d = DeviceProblem(p)
    cases = [dict(plan=s.SPMV_PLAN_MERGE, items_per_chunk=i) for i in (0, 1, 7, 255, 256, 257, 258, 1023, 1024, 8192)] + [dict(plan=s.SPMV_PLAN_TWOPHASE)]
    for params in cases:
        A = d.matrix(params)
        for _ in range(4):
            y = d.run(A)
            assert np.array_equal(y.astype(np.float64), y_ref), (name, params)
        A.close()
    for _ in range(3):
        y = d.y0.clone()
        s.check(s.spmv_csr_run_static(p.m, p.n, p.nnz, d.rowptr.data_ptr(), d.colidx.data_ptr(), d.vals.data_ptr(), DTYPE_CODE[dtype],
                                      d.x.data_ptr(), y.data_ptr(), p.alpha, p.beta))
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy().astype(np.float64), y_ref), name


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("plan,length,rows", [(s.SPMV_PLAN_MERGE, 300, 9000), (s.SPMV_PLAN_TWOPHASE, 700, 8300)])
def test_most_chunks_cut_a_row(plan, length, rows, dtype):
    """12 * (cuts - 600) > chunks: the pieces are left to a kernel behind the chunks, in the handle and (2048 steps a chunk, 1024
    chunks or more) without one.  Repeated, on a stream, and replayed from a graph."""
    lens = np.full(rows, length)
    lens[100:300], lens[rows // 2] = 1, 9 * length
    p = w.exact_integer(lens, 70000, seed=31, dtype=dtype, alpha=2.0, beta=-1.0)
    row, nz = oracle.merge_path(p.rowptr, 2048) if plan == s.SPMV_PLAN_MERGE else oracle.merge_path_snapped(p.rowptr, 8192, 512)
    inside = (row < p.m) & (nz > p.rowptr[np.minimum(row, p.m - 1)])
    cuts = int((inside & (lens[np.minimum(row, p.m - 1)] > (256 if plan == s.SPMV_PLAN_MERGE else 512))).sum())
    assert 12 * (cuts - 600) > row.size - 1
    y_ref, _ = oracle.spmv_problem(p)
    d = DeviceProblem(p)
    A = d.matrix(dict(plan=plan))
    for _ in range(3):
        assert np.array_equal(d.run(A).astype(np.float64), y_ref)
    y = d.y0.clone()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=torch.cuda.Stream()):
        A.run(d.x, y, p.alpha, p.beta, torch.cuda.current_stream().cuda_stream)
    for _ in range(3):
        y.copy_(d.y0)
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy().astype(np.float64), y_ref)
        assert np.array_equal(d.run(A).astype(np.float64), y_ref)
    A.close()
    y = d.y0.clone()
    s.check(s.spmv_csr_run_static(p.m, p.n, p.nnz, d.rowptr.data_ptr(), d.colidx.data_ptr(), d.vals.data_ptr(), DTYPE_CODE[dtype],
                                  d.x.data_ptr(), y.data_ptr(), p.alpha, p.beta))
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy().astype(np.float64), y_ref)


def test_cut_rows_replayed_from_a_graph():
    p = w.exact_integer([4] * 3000 + [20000, 600, 9000], 30000, seed=12)
    y_ref, _ = oracle.spmv_problem(p)
    d = DeviceProblem(p)
    for plan in (s.SPMV_PLAN_MERGE, s.SPMV_PLAN_TWOPHASE):
        A = d.matrix(dict(plan=plan))
        y = torch.zeros(p.m, device="cuda")
        A.run(d.x, y)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=torch.cuda.Stream()):
            for _ in range(3):
                A.run(d.x, y, 1.0, 0.0, torch.cuda.current_stream().cuda_stream)
        for _ in range(3):
            y.fill_(7.0)
            g.replay()
            torch.cuda.synchronize()
            assert np.array_equal(y.cpu().numpy().astype(np.float64), y_ref)
            A.run(d.x, y)
            torch.cuda.synchronize()
            assert np.array_equal(y.cpu().numpy().astype(np.float64), y_ref)
        A.close()


@pytest.mark.parametrize("length", [1, 4, 7, 8, 12, 16, 20, 64, 100, 256, 512])
def test_two_pass_rows_of_one_length(length):
    """Chunks of rows of one length take more lanes per row where that length is a multiple of four; one odd row in between."""
    for lens in ([length] * (20000 // length + 3), [length] * 501 + [length + 1] + [length] * 700):
        p = w.exact_integer(lens, 9000, seed=length, alpha=1.0, beta=1.0)
        y_ref, _ = oracle.spmv_problem(p)
        d = DeviceProblem(p)
        A = d.matrix(dict(plan=s.SPMV_PLAN_TWOPHASE))
        assert np.array_equal(d.run(A).astype(np.float64), y_ref), (length, len(lens))
        A.close()


@pytest.mark.parametrize("plan", [s.SPMV_PLAN_MERGE, s.SPMV_PLAN_TWOPHASE])
def test_second_stream_as_soon_as_the_first_run_reports_completion(plan):
    """One handle on two streams, ordered by nothing but the refusals: the second stream's run is asked for until it is no
    longer refused, so all that stands between two runs that share the plan's scratch is the query of the first one's event.
    Different inputs on the two streams; integers, so both results equal the oracle's bit for bit, every time."""
    lens = [9] * 60000 + [30000, 700, 0, 5000] + [9] * 60000
    p = w.exact_integer(lens, 120000, seed=21, alpha=1.0, beta=1.0)
    d = DeviceProblem(p)
    A = d.matrix(dict(plan=plan))
    x2 = (-2 * p.x).astype(np.float32)
    y1_ref, _ = oracle.spmv_problem(p)
    y2_ref, _ = oracle.spmv_csr("f32", p.m, p.n, p.rowptr, p.colidx, p.vals, x2, p.y0, p.alpha, p.beta)
    x2_t = torch.from_numpy(x2).cuda()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    refused = 0
    for rep in range(20):
        y1, y2 = d.y0.clone(), d.y0.clone()
        torch.cuda.synchronize()
        s.check(s.spmv_csr_run(A.handle, d.x.data_ptr(), y1.data_ptr(), p.alpha, p.beta, s1.cuda_stream))
        deadline = time.monotonic() + 20
        while True:
            status = s.spmv_csr_run(A.handle, x2_t.data_ptr(), y2.data_ptr(), p.alpha, p.beta, s2.cuda_stream)
            if status != s.SPMV_ERR_BUSY:
                break
            refused += 1
            assert time.monotonic() < deadline
        s.check(status)
        torch.cuda.synchronize()
        assert np.array_equal(y1.cpu().numpy().astype(np.float64), y1_ref), rep
        assert np.array_equal(y2.cpu().numpy().astype(np.float64), y2_ref), rep
    assert refused > 0
    A.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_cut_rows_of_the_two_pass_plan_on_groups(dtype):
    """Group-aligned matrices with rows of more than 512 groups: the chunks then count groups, and so do the cuts."""
    groups = {"around_the_snap": [511, 512, 513, 0, 3, 700] * 30, "long_rows_between_short_ones": [5] * 300 + [3000, 0, 20000] + [1] * 500 + [8193, 2, 9000],
              "starts_and_ends_long": [9000] + [2] * 5000 + [9000]}
    for name, per_row in groups.items():
        p = w.exact_integer([8 * g for g in per_row], 200000, seed=13, dtype=dtype, alpha=2.0, beta=-1.0)
        first = np.random.default_rng(14).integers(0, p.n // 8, p.nnz // 8)
        p.colidx[:] = (8 * first[:, None] + np.arange(8)).reshape(-1)
        y_ref, _ = oracle.spmv_problem(p)
        d = DeviceProblem(p)
        A = d.matrix(dict(plan=s.SPMV_PLAN_TWOPHASE))
        assert A.info.tp_group == 8
        got = A.analysis()
        cut = got["tp_nz"] > p.rowptr[np.minimum(got["tp_row"], p.m)] // 8
        assert cut[got["tp_row"] < p.m].sum() >= 2, name           # some chunks do cut a row
        for rep in range(4):
            y = d.run(A)
            assert np.array_equal(y.astype(np.float64), y_ref), (name, rep)
        A.close()
