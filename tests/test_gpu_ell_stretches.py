"""GPU: ELL rows of up to 64 slots at the widths where a lane's share of a row changes, with padding anywhere in a row.  What padding
slots hold, and x where only padding would read it, is NaN; integers elsewhere, so the result equals the oracle's bit for bit."""
import numpy as np
import pytest
import torch

import paper_2603_07169_amd as s
import workloads as w
from gpu_util import DTYPE_CODE, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("width", [1, 3, 4, 5, 8, 9, 12, 13, 16, 24, 25, 28, 32, 40, 48, 52, 64])
def test_padding_counts_for_nothing(width, dtype, offset):
    rng = np.random.Generator(np.random.Philox(key=[np.uint64(width), np.uint64(offset)]))
    for m in (1, 63, 515):
        n = 300
        cols = rng.integers(1, n, (m, width)).astype(np.int32)
        vals = rng.integers(-4, 5, (m, width)).astype(np.float32)
        x = rng.integers(-4, 5, n).astype(np.float32)
        y0 = rng.integers(-4, 5, m).astype(np.float32)
        pad = rng.random((m, width)) < 0.3
        pad[m // 2] = True                        # a row of padding only
        want = (np.where(pad, 0.0, vals.astype(np.float64) * x[cols].astype(np.float64))).sum(1) + 2.0 * y0
        cols[pad] = -1
        vals[pad] = np.nan
        x[0] = np.nan                             # no entry has column 0
        if dtype == "bf16":
            vals, x = w.f32_to_bf16_bits(np.where(np.isnan(vals), 0, vals)), w.f32_to_bf16_bits(np.where(np.isnan(x), 0, x))
            vals[pad], x[0] = 0x7FC0, 0x7FC0
        ci_t, v_t, x_t, y = to_dev(cols.reshape(-1), offset), to_dev(vals.reshape(-1), offset), to_dev(x), to_dev(y0)
        s.check(s.spmv_ell_run(m, n, width, ci_t.data_ptr(), v_t.data_ptr(), DTYPE_CODE[dtype], x_t.data_ptr(), y.data_ptr(), 1.0, 2.0))
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy().astype(np.float64), want), (width, dtype, offset, m)
