"""GPU: the multiply pass on groups of eight at pieces of fewer trips (of 1024 slots) than it takes at once (eight in bf16, four in FP32), of
whole rounds, and with a remainder of two trips or fewer, of up to half a round and of more; integers, so every order of the sums gives the
same bits."""
import numpy as np
import pytest
import torch

import paper_2603_07169_amd as s
import workloads as w
from gpu_util import DeviceProblem, reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("groups", [1, 1000, 1025, 2 * 1024 + 4, 5 * 1024, 8 * 1024, 9 * 1024 + 700, 12 * 1024 + 1, 16 * 1024, 3 * 16384 + 4100])
def test_pieces_of_every_length(groups, dtype):
    n = 8 * 500                                  # one column block: pieces of at most 2048 groups of four slots, eight trips
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
    trips = np.diff(A.analysis()["tp_piece_g"]) / 256
    assert A.info.tp_group == 8 and groups / 1024 <= trips.sum() < groups / 1024 + 1 and trips.max() <= 8
    want, _ = reference(p)
    assert np.array_equal(d.run(A).astype(np.float64), want)
    A.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("trips", [8.5, 10.9, 12, 12.6, 15.9])
def test_pieces_of_more_trips_than_a_round(trips, dtype):
    """Matrices large enough for the rule to make pieces of 8 to 16 trips (a piece for every workgroup that is held at once): a second round
    in bf16, and after it nothing; made and checked on the GPU."""
    resident = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    per_row, n = 4, 8 * 500
    m = int(trips * 1024 * resident / per_row)
    g = torch.Generator(device="cuda").manual_seed(int(10 * trips))
    ints = lambda *k: torch.randint(-3, 4, k, generator=g, device="cuda").float()
    first = torch.randint(0, n // 8, (m * per_row,), generator=g, device="cuda", dtype=torch.int32)
    colidx = (8 * first[:, None] + torch.arange(8, dtype=torch.int32, device="cuda")).view(-1)
    vals, x, y0 = ints(m * per_row * 8), ints(n), ints(m)
    want = (vals.view(-1, 8) * x.view(-1, 8)[first.long()]).view(m, -1).sum(1) + 2.0 * y0
    rowptr = torch.arange(m + 1, dtype=torch.int32, device="cuda") * (8 * per_row)
    store = torch.bfloat16 if dtype == "bf16" else torch.float32
    vals, x = vals.to(store), x.to(store)
    A = s.CsrMatrix(m, n, rowptr, colidx, vals, s.SPMV_BF16 if dtype == "bf16" else s.SPMV_F32, dict(plan=s.SPMV_PLAN_TWOPHASE))
    print("case", trips, dtype, colidx.numel(), A.info.tp_piece_groups / 256, flush=True)
    assert A.info.tp_group == 8 and trips - 0.02 <= A.info.tp_piece_groups / 256 <= trips + 0.3
    y = y0.clone()
    A.run(x, y, 1.0, 2.0, None)
    torch.cuda.synchronize()
    assert torch.equal(y, want)
    A.close()
