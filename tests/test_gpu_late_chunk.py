"""A default all-gather or grouped plan of several waves whose first chunk lands last: the
tiles that wait for it hold up nothing else. The late chunk is one copy of 128 MiB, which
takes an engine milliseconds; the other tiles are half a millisecond of work."""
import pytest

import paper_2601_20595_amd as csg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("op", ["ag", "grouped"])
def test_tiles_that_wait_for_a_late_chunk_hold_up_no_other(op):
    late, rest, N, K = 8192, 16384, 1024, 8192          # 32 and 64 row tiles, 4 column tiles
    print("late chunk", op, flush=True)
    chunks = [(0, late, 1, 0, 0), (late, late + rest, 0, 0, 1)]
    plan = csg.Plan(op, late + rest, N, K, "bf16", "bf16", csg.Schedule.create(chunks, [0, 1]),
                    group_rows=[late + rest] if op == "grouped" else None, cfg={"trace": 1, "timeout_ms": 1000})
    assert plan.info.n_units == plan.info.n_tiles == 384 > plan.info.num_workgroups >= 256
    a = torch.zeros((late + rest, K), device=DEV, dtype=torch.bfloat16)
    b = torch.zeros((1, N, K) if op == "grouped" else (N, K), device=DEV, dtype=torch.bfloat16)
    landing, c = a.clone(), torch.empty((late + rest, N), device=DEV, dtype=torch.bfloat16)
    st, cp = torch.cuda.Stream(), torch.cuda.Stream()
    for _ in range(2):                                  # (the first call loads the kernel)
        torch.cuda.synchronize()
        (plan.ag_gemm if op == "ag" else plan.grouped_gemm)(landing, a, b, c, "overlap", st, cp)
        plan.check()
        torch.cuda.synchronize()
    t = plan.trace()
    waits = t["raster"] // plan.info.n_tiles_n < late // 256
    assert waits.sum() == 128 and (~waits).sum() == 256
    assert t["t_end"][~waits].max() < t["t_start"][waits].min()
    plan.close()
