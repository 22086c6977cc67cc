"""GPU: ELL rows whose tiles are cut to whole sweeps of the row phase, at the widths and row counts where the cut changes;
integers, so the result equals the oracle's bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_07169_amd as s
import workloads as w
from gpu_util import DTYPE_CODE, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("width,most", [(1, 3 << 19), (2, 3 << 17)])
def test_narrow_rows_on_both_sides_of_the_rule(width, most, dtype):
    """Rows of one or two slots: up to `most` of them a lane reads its row itself, beyond that they go through LDS."""
    for m in (most, most + 1):
        p = w.exact_integer(np.arange(m) % (width + 1), 5000, seed=width, dtype=dtype, alpha=1.0, beta=2.0)
        y_ref, _ = oracle.spmv_problem(p)
        wd, ci, vals = w.to_ell(p)
        ci_t, v_t, x_t, y = to_dev(ci), to_dev(vals), to_dev(p.x), to_dev(p.y0)
        s.check(s.spmv_ell_run(p.m, p.n, wd, ci_t.data_ptr(), v_t.data_ptr(), DTYPE_CODE[dtype], x_t.data_ptr(), y.data_ptr(), 1.0, 2.0))
        torch.cuda.synchronize()
        assert wd == width and np.array_equal(y.cpu().numpy().astype(np.float64), y_ref), m


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("width", [1, 15, 16, 17, 27, 31, 32, 33, 43, 48, 49, 63, 64])
def test_tiles_of_every_width(width, dtype):
    for m in (1, 127, 129, 145, 64 * 24 + 3):     # 8 dies: fewer tiles than dies, and a remainder over them
        lens = np.minimum(np.arange(m) % (width + 1) + (np.arange(m) % 3 == 0) * width, width)
        lens[m // 2] = width
        p = w.exact_integer(lens, 5000, seed=width, dtype=dtype, alpha=1.0, beta=2.0)
        y_ref, _ = oracle.spmv_problem(p)
        wd, ci, vals = w.to_ell(p)
        assert wd == width
        ci_t, v_t, x_t, y = to_dev(ci), to_dev(vals), to_dev(p.x), to_dev(p.y0)
        s.check(s.spmv_ell_run(p.m, p.n, wd, ci_t.data_ptr(), v_t.data_ptr(), DTYPE_CODE[dtype], x_t.data_ptr(), y.data_ptr(), 1.0, 2.0))
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy().astype(np.float64), y_ref), (width, m)


def test_coo_of_more_than_16384_stretches():
    """Beyond 16 M entries a workgroup takes two stretches of the coordinate kernel."""
    p = w.exact_integer([8] * 2_200_000, 4096, seed=3)
    y_ref, _ = oracle.spmv_problem(p)
    row, col, vals = (to_dev(a) for a in w.to_coo(p))
    x_t, y = to_dev(p.x), torch.zeros(p.m, device="cuda")
    s.check(s.spmv_coo_run(p.m, p.n, p.nnz, row.data_ptr(), col.data_ptr(), vals.data_ptr(), s.SPMV_F32, x_t.data_ptr(), y.data_ptr(), 1.0, 0.0))
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy().astype(np.float64), y_ref)
