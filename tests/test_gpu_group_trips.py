"""GPU: the multiply pass on groups of eight at pieces of fewer trips than it takes at once, of whole rounds, and of every remainder;
integers, so the result equals the oracle's bit for bit."""
import numpy as np
import pytest

import paper_2603_07169_amd as s
import workloads as w
from gpu_util import DeviceProblem, reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("groups", [1, 1000, 1025, 2 * 1024 + 4, 5 * 1024, 8 * 1024, 9 * 1024 + 700, 12 * 1024 + 1, 16 * 1024, 3 * 16384 + 4100])
def test_pieces_of_every_length(groups, dtype):
    n = 8 * 500                                  # one column block: pieces of up to 16384 groups of slots
    rng = np.random.Generator(np.random.Philox(key=[np.uint64(groups), np.uint64(0)]))
    per_row = 4 if groups >= 4 else 1
    m = -(-groups // per_row)
    counts = np.full(m, per_row)
    counts[-1] -= per_row * m - groups
    first = rng.integers(0, n // 8, groups)
    colidx = (8 * first[:, None] + np.arange(8)).reshape(-1).astype(np.int32)
    rowptr = np.concatenate([[0], np.cumsum(8 * counts)]).astype(np.int32)
    ints = lambda k: rng.integers(-3, 4, k).astype(np.float32)
    vals, x, y0 = ints(colidx.size), ints(n), ints(m)
    if dtype == "bf16":
        vals, x = w.f32_to_bf16_bits(vals), w.f32_to_bf16_bits(x)
    p = w.CsrProblem(f"groups_{groups}", dtype, m, n, rowptr, colidx, vals, x, y0, 1.0, 2.0)
    d = DeviceProblem(p)
    A = d.matrix(dict(plan=s.SPMV_PLAN_TWOPHASE))
    assert A.info.tp_group == 8
    want, _ = reference(p)
    assert np.array_equal(d.run(A).astype(np.float64), want)
    A.close()
