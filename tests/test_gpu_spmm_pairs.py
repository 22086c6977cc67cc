"""GPU: the pairs form of A (sparse times dense with B of at most 2048 rows, handle analysed with prepare_spmm): its layout bit
for bit against the oracle's, and products from it at the edges of its groups (32 rows), blocks (4 entries), ordered
stretches (256 entries) and slices (16 columns).  Every product is asked which kernel it takes."""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_07169_amd as s
import workloads as w
from gpu_util import DeviceProblem, to_dev
from test_gpu_spmm import TOLS, b_tensor, rand, rand_b

pytestmark = pytest.mark.gpu
PAIRS, PACKED, PLAIN = "spmm_pair_kernel", "spmm_packed_kernel", "spmm_csr_kernel"


def buffers(p, B, C0, ldb, ldc, offset=0):
    """B and C as views of wider allocations that start `offset` elements in; what is not theirs holds 7."""
    K = B.shape[1]
    Bbuf = torch.full((p.n * ldb + offset,), 7, dtype=torch.int16 if B.dtype == np.uint16 else torch.float32, device="cuda")
    Cbuf = torch.full((p.m * ldc + offset,), 7.0, dtype=torch.float32, device="cuda")
    Bt, C_all = Bbuf[offset:].view(p.n, ldb)[:, :K], Cbuf[offset:].view(p.m, ldc)
    Bt.copy_(b_tensor(B))
    C_all[:, :K].copy_(torch.from_numpy(C0))
    return Bt, C_all


def kernel_of(A, Bt, Ct):
    return s.spmm_csr_kernel_name(A.handle, Bt.data_ptr(), Bt.stride(0), Ct.data_ptr(), Ct.stride(0), Bt.shape[1])


def check_product(A, p, K, ldb, ldc, alpha, beta, kernel=PAIRS, offset=0, seed=0):
    B, C0 = rand_b(p, K, seed), rand((p.m, K), seed + 1)
    if beta == 0:
        C0[:] = np.nan                                              # not read
    Bt, C_all = buffers(p, B, C0, ldb, ldc, offset)
    Ct = C_all[:, :K]
    assert kernel_of(A, Bt, Ct) == kernel, (p.name, K, ldb, ldc, offset)
    print("case spmm pairs", p.name, p.m, p.dtype, K, ldb, ldc, offset, alpha, beta, flush=True)
    A.spmm(Bt, Ct, alpha, beta)
    torch.cuda.synchronize()
    C_ref, S = oracle.spmm_csr(p.m, p.n, p.rowptr, p.colidx, p.vals, B, C0, alpha, beta)
    bound = TOLS[p.dtype] * (abs(alpha) * S + (np.abs(np.float64(np.float32(beta)) * C0) if beta != 0 else 0.0))
    err = np.abs(Ct.cpu().numpy().astype(np.float64) - C_ref)
    bad = np.argwhere(~(err <= bound))
    assert bad.size == 0, (p.name, K, bad[:3].tolist(), err[tuple(bad[0])], bound[tuple(bad[0])])
    assert bool((C_all[:, K:] == 7.0).all())                        # the columns behind C's are not touched


def expected_forms(p):
    """The packed copy's and the pairs form's layouts as the oracle has them, or None."""
    packed_rows = oracle.spmm_row_order(p.rowptr)
    packed_desc, packed_blocks = oracle.spmm_packed_layout(p.rowptr, packed_rows)
    if not oracle.spmm_packed_choice(p.nnz, packed_blocks):
        return None, None
    rows = oracle.spmm_pair_row_order(p.rowptr)
    desc, blocks = oracle.spmm_pair_layout(p.rowptr, rows)
    return packed_blocks, (rows, desc, blocks) if oracle.spmm_pair_choice(p.m, p.n, blocks, packed_desc) else None


LAYOUTS = {
    "benchmark": lambda dt: w.density_random(1 << 13, 2048, 0.01, dtype=dt),
    "odd_rows": lambda dt: w.density_random(4099, 2047, 0.01, dtype=dt),
    "stretches": lambda dt: w.from_row_lengths([255] * 16 + [256] * 16 + [257] * 16 + [600] * 17, 2048, seed=2, dtype=dt, allow_dup=True, sort_cols=False),
    "long_equal": lambda dt: w.from_row_lengths([1100] * 31 + [1024] * 33, 300, seed=3, dtype=dt, allow_dup=True),
    "short": lambda dt: w.from_row_lengths(list(np.arange(63) % 5 + 12), 20, seed=4, dtype=dt),
    "empty_rows": lambda dt: w.from_row_lengths(([16] * 25 + [0] * 7) * 6, 500, seed=5, dtype=dt),
    "uniform_spread": lambda dt: w.from_row_lengths(np.random.default_rng(6).integers(1, 200, 5000), 2048, seed=6, dtype=dt, allow_dup=True),
    "skewed_refused": lambda dt: w.from_row_lengths([27, 28, 29, 30] * 9, 2048, seed=7, dtype=dt),
    "wide_refused": lambda dt: w.uniform_rows(600, 2049, 20, dtype=dt),
    "unpacked": lambda dt: w.from_row_lengths([5] * 31, 2048, seed=8, dtype=dt),
}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("name", LAYOUTS)
def test_layout_read_back_equals_the_oracles(name, dtype):
    p = LAYOUTS[name](dtype)
    A = DeviceProblem(p).matrix(dict(prepare_spmm=1))
    packed_blocks, pairs = expected_forms(p)
    assert (pairs is None) == (name in ("skewed_refused", "wide_refused", "unpacked"))
    assert A.info.spmm_prepared == (1 if packed_blocks is None else 2)
    got = A.analysis()
    if pairs is None:
        assert A.info.spmm_pair_blocks == 0 and "spmm_pair_ent" not in got
    else:
        rows, desc, blocks = pairs
        assert A.info.spmm_pair_blocks == blocks
        assert np.array_equal(got["spmm_pair_rows"], rows) and np.array_equal(got["spmm_pair_desc"], desc)
        off, src = oracle.spmm_pair_pack(p.rowptr, p.colidx, rows, desc)
        ent = got["spmm_pair_ent"].reshape(-1, 4)
        assert np.array_equal(got["spmm_pair_src"], src)
        assert np.array_equal(ent[:, :2].reshape(-1).astype(np.int32), off)
        vals = p.vals if dtype == "f32" else w.bf16_bits_to_f32(p.vals)
        assert np.array_equal(ent[:, 2:].reshape(-1).view(np.float32), np.where(src >= 0, vals[np.maximum(src, 0)], np.float32(0)))
    A.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_columns_in_one_slot(dtype):
    """Every column in one slot of the LDS banks: no order avoids the conflicts."""
    p = w.from_row_lengths([14] * 80, 2048, seed=3, dtype=dtype)
    p.colidx[:] = p.colidx // 8 * 8
    A = DeviceProblem(p).matrix(dict(prepare_spmm=1))
    rows, desc, blocks = expected_forms(p)[1]
    assert np.array_equal(A.analysis()["spmm_pair_src"], oracle.spmm_pair_pack(p.rowptr, p.colidx, rows, desc)[1])
    check_product(A, p, 33, 33, 33, 1.0, 1.0)
    A.close()


EDGES = [  # row lengths, columns, ldb, ldc
    (list(np.arange(63) % 5 + 12), [(1, 1, 1), (15, 15, 17), (16, 17, 16), (17, 21, 18), (33, 33, 33), (100, 101, 103)]),
    (list(np.arange(64) % 5 + 12), [(1, 3, 5), (16, 16, 19), (47, 47, 49), (1025, 1028, 1028)]),
    ([13] * 31, [(1, 1, 1), (20, 21, 21), (49, 49, 49)]),
    ([12] * 32 + [9] * 30 + [8, 7], [(31, 31, 31), (65, 65, 66)]),
    (list(np.arange(64) % 5 + 28), [(777, 777, 779), (1025, 1025, 1028)]),
    (list(np.arange(65) % 5 + 28), [(1025, 1028, 1028), (2049, 2049, 2050)]),      # one row in the last group, one column in the last slice
    ([255] * 16 + [256] * 16 + [257] * 16 + [600] * 16, [(2049, 2049, 2051)]),     # one, two and three stretches
    (([16] * 25 + [0] * 7) * 6, [(17, 17, 17), (130, 131, 131)]),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("edge", range(len(EDGES)))
def test_edges(edge, dtype):
    lens, shapes = EDGES[edge]
    p = w.from_row_lengths(lens, 2048, seed=edge, dtype=dtype, allow_dup=True, sort_cols=False)
    A = DeviceProblem(p).matrix(dict(prepare_spmm=1))
    assert A.info.spmm_pair_blocks > 0
    for K, ldb, ldc in shapes:
        for alpha, beta, offset in ((1.0, 0.0, 0), (-1.5, 0.5, 3)):
            check_product(A, p, K, ldb, ldc, alpha, beta, offset=offset, seed=K)
    A.close()


def test_more_slices_than_compute_units_and_aligned_rows():
    p = w.from_row_lengths([20] * 2400, 100, seed=4)
    A = DeviceProblem(p).matrix(dict(prepare_spmm=1))
    check_product(A, p, 4130, 4130, 4130, 1.0, 0.0, seed=2)
    check_product(A, p, 4130, 4132, 4132, 2.0, 1.0, seed=3)
    A.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("m,ldc", [(49, (1 << 22) + 5), (160, (1 << 22) - 1), (300, (1 << 22) - 1)])
def test_rows_of_c_far_apart(m, ldc, dtype):
    """Leading dimension from 2^22 on, and C of more than 4 GiB: offsets into C take 64 bits; C of more than 2 GiB: they fill 32."""
    p = w.from_row_lengths(list(np.arange(m) % 5 + 12), 40, seed=5, dtype=dtype, allow_dup=True)
    A = DeviceProblem(p).matrix(dict(prepare_spmm=1))
    B = rand_b(p, 20, 1)
    C0 = rand((p.m, 20), 2)
    for beta in (0.0, 0.5):
        C_all = torch.empty(p.m, ldc, dtype=torch.float32, device="cuda")
        Bt, Ct = b_tensor(B).cuda(), C_all[:, :20]
        Ct.copy_(torch.from_numpy(C0))
        C_all[:, 20:36] = 7.0
        assert kernel_of(A, Bt, Ct) == PAIRS
        print("case spmm far apart", m, ldc, dtype, beta, flush=True)
        A.spmm(Bt, Ct, 2.0, beta)
        torch.cuda.synchronize()
        C_ref, S = oracle.spmm_csr(p.m, p.n, p.rowptr, p.colidx, p.vals, B, C0, 2.0, beta)
        assert np.all(np.abs(Ct.cpu().numpy() - C_ref) <= TOLS[dtype] * (2.0 * S + np.abs(beta * C0)))
        assert bool((C_all[:, 20:36] == 7.0).all())
    A.close()


def test_rows_of_b_that_no_entry_names_stay_out():
    """Padding reads zero rows: infinities and NaN in rows of B without an entry do not reach C."""
    p = w.from_row_lengths(list(np.arange(63) % 5 + 12), 1000, seed=9, allow_dup=True)
    p.colidx[:] = p.colidx // 2 * 2
    A = DeviceProblem(p).matrix(dict(prepare_spmm=1))
    B = rand((p.n, 33), 1)
    C_ref, S = oracle.spmm_csr(p.m, p.n, p.rowptr, p.colidx, p.vals, B)
    B[1::4], B[3::4] = np.inf, np.nan
    Bt, Ct = torch.from_numpy(B).cuda(), torch.zeros(p.m, 33, device="cuda")
    assert kernel_of(A, Bt, Ct) == PAIRS
    A.spmm(Bt, Ct)
    torch.cuda.synchronize()
    assert np.all(np.abs(Ct.cpu().numpy() - C_ref) <= TOLS["f32"] * S)
    A.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_both_forms_of_one_handle(dtype):
    """A handle that holds both takes few columns from the packed copy and many from the pairs form; rows of very different
    lengths stay with the packed copy."""
    p = w.density_random(1 << 14, 2048, 0.01, dtype=dtype)
    A = DeviceProblem(p).matrix(dict(prepare_spmm=1))
    check_product(A, p, 16, 16, 16, 1.0, 0.5, kernel=PACKED)
    check_product(A, p, 65, 65, 65, 1.0, 0.5, kernel=PAIRS)
    Bt, Ct = torch.zeros(p.n, 4096, device="cuda"), torch.zeros(p.m, 4096, device="cuda")
    assert kernel_of(A, Bt, Ct) == PAIRS
    A.close()
    lens = np.where(np.arange(4096) % 200 == 0, 600, 20)
    q = w.from_row_lengths(lens, 2048, seed=3, dtype=dtype, allow_dup=True)
    A = DeviceProblem(q).matrix(dict(prepare_spmm=1))
    assert A.info.spmm_pair_blocks > 0
    check_product(A, q, 64, 64, 64, 1.0, 0.0, kernel=PACKED)
    A.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_refreshed_values_and_read_back(dtype):
    """After new values the products use them once the handle was told, and both forms read back hold them."""
    p = w.density_random(300, 900, 0.02, dtype=dtype)
    d = DeviceProblem(p)
    A = d.matrix(dict(prepare_spmm=1))
    assert A.info.spmm_prepared == 2 and A.info.spmm_pair_blocks > 0
    before = A.analysis()
    q = w.density_random(300, 900, 0.02, dtype=dtype)
    q.vals = q.vals[::-1].copy()
    d.vals.copy_(to_dev(q.vals).view(d.vals.dtype))
    now = A.analysis()
    for key in ("spmm_val", "spmm_pair_ent"):
        assert np.array_equal(now[key], before[key])                # as they were at analyze time
    A.refresh_values()
    torch.cuda.synchronize()
    check_product(A, q, 777, 777, 777, 1.0, 0.0, kernel=PAIRS)
    check_product(A, q, 40, 40, 40, 1.0, 0.0, kernel=PACKED)
    fresh = DeviceProblem(q)
    F = fresh.matrix(dict(prepare_spmm=1))
    now, want = A.analysis(), F.analysis()
    for key in ("spmm_val", "spmm_pair_ent", "spmm_pair_src"):
        assert np.array_equal(now[key], want[key])
    A.close()
    F.close()


def test_replayed_from_a_graph():
    p = w.density_random(1 << 12, 2048, 0.01)
    A = DeviceProblem(p).matrix(dict(prepare_spmm=1))
    B = torch.from_numpy(rand((p.n, 65), 1)).cuda()
    C, want = torch.zeros(p.m, 65, device="cuda"), torch.zeros(p.m, 65, device="cuda")
    assert kernel_of(A, B, C) == PAIRS
    A.spmm(B, want)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=torch.cuda.Stream()):
        A.spmm(B, C, 1.0, 0.0, torch.cuda.current_stream().cuda_stream)
    for _ in range(3):
        C.fill_(5.0)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(C, want)
        A.spmm(B, want)
        torch.cuda.synchronize()
    A.close()
