"""GPU parity of the sparse-times-dense product from the pairs form of A (B of at most 2048 rows, handle analysed with
prepare_spmm): edges of its groups (32 rows), blocks (4 entries), ordered stretches (256 entries) and slices (16 columns)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_07169_amd as s
import workloads as w
from gpu_util import DeviceProblem, to_dev
from test_gpu_spmm import TOLS, b_tensor, check, rand, rand_b

pytestmark = pytest.mark.gpu


def product(A, p, B, C0, alpha, beta, ld=None):
    K = B.shape[1]
    Bt = b_tensor(B).cuda()
    Cbuf = torch.zeros(p.m * (ld or K), dtype=torch.float32, device="cuda")
    Ct = Cbuf.view(p.m, ld or K)[:, :K]
    Ct.copy_(torch.from_numpy(C0))
    A.spmm(Bt, Ct, alpha, beta)
    torch.cuda.synchronize()
    return Ct.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("lens", [[5] * 31, [4] * 32 + [3], list(range(66)), [27, 28, 29, 30] * 9, [255, 256, 257] * 11 + [600, 513],
                                  [0] * 40 + [1], [1024] * 3 + [2] * 61], ids=str)
def test_edges(lens, dtype):
    p = w.from_row_lengths(lens, 2048, seed=len(lens), dtype=dtype, allow_dup=True, sort_cols=False)
    for K in (1, 16, 33, 100):
        for alpha, beta in ((1.0, 0.0), (-1.5, 0.5)):
            check(p, K, alpha=alpha, beta=beta, seed=K)


def test_one_slot_for_all_columns_and_many_slices():
    """Every column in one slot of the LDS banks (no order avoids the conflicts), and more slices than compute units."""
    p = w.from_row_lengths([9] * 70, 2048, seed=3)
    p.colidx[:] = p.colidx // 8 * 8
    check(p, 24, alpha=1.0, beta=1.0, seed=1)
    check(w.from_row_lengths([20] * 600, 100, seed=4), 4130, seed=2)


def test_rows_of_c_far_apart():
    """Leading dimension of 2^22 and more: offsets into C take 64 bits."""
    p = w.from_row_lengths([3, 0, 17], 40, seed=5)
    A = DeviceProblem(p)
    M = A.matrix(dict(prepare_spmm=1))
    B, C0 = rand((p.n, 20), 1), rand((p.m, 20), 2)
    for beta in (0.0, 0.5):
        C_ref, S = oracle.spmm_csr(p.m, p.n, p.rowptr, p.colidx, p.vals, B, C0, 2.0, beta)
        C = product(M, p, B, C0, 2.0, beta, ld=(1 << 22) + 4)
        assert np.all(np.abs(C - C_ref) <= TOLS["f32"] * (2.0 * S + np.abs(beta * C0)))
    M.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_refreshed_values_and_read_back(dtype):
    """After new values the product uses them once the handle was told, and the packed copy read back holds them."""
    p = w.density_random(300, 900, 0.02, dtype=dtype)
    d = DeviceProblem(p)
    A = d.matrix(dict(prepare_spmm=1))
    assert A.info.spmm_prepared == 2
    before = A.analysis()["spmm_val"].copy()
    q = w.density_random(300, 900, 0.02, dtype=dtype)
    q.vals = q.vals[::-1].copy()
    d.vals.copy_(to_dev(q.vals).view(d.vals.dtype))
    assert np.array_equal(A.analysis()["spmm_val"], before)      # as they were at analyze time
    A.refresh_values()
    torch.cuda.synchronize()
    B, C0 = rand_b(q, 40, 3), rand((q.m, 40), 4)
    C_ref, S = oracle.spmm_csr(q.m, q.n, q.rowptr, q.colidx, q.vals, B, C0, 1.0, 0.0)
    assert np.all(np.abs(product(A, q, B, C0, 1.0, 0.0) - C_ref) <= TOLS[dtype] * S)
    fresh = DeviceProblem(q)
    F = fresh.matrix(dict(prepare_spmm=1))
    assert np.array_equal(A.analysis()["spmm_val"], F.analysis()["spmm_val"])
    A.close()
    F.close()
