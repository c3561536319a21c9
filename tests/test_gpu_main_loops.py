"""GPU parity of the bf16 main loops at the edges of their pipelines: one K step (the ring
is never full), two, three and more, slices of a single step, tiles with one valid row or
a few valid columns. Integer inputs, so every sum is exact in fp32 and the output must
match the oracle bit for bit."""
import numpy as np
import pytest

import oracle
import paper_2601_20595_amd as csg
import seeded_inputs as si

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from gpu_util import bf16_rne_of_f64, out_to_f64, run_ag, run_rs

TILES = [(256, 256)]


@pytest.mark.parametrize("tile", TILES, ids=lambda t: "%dx%d" % t)
@pytest.mark.parametrize("steps,split", [(1, 1), (2, 1), (3, 1), (4, 1), (9, 1), (3, 3), (7, 2)])
@pytest.mark.parametrize("op", ["ag", "rs"])
def test_pipeline_edges_bit_exact(tile, steps, split, op):
    W, r, S, Q = 2, 1, 257, 1                     # 514 rows: the last row tile holds a row or two
    N, K = 256 + 4, 64 * steps                    # the last column tile holds four columns
    print("main loop", tile, steps, split, op, flush=True)
    w = si.Workload(131, "loop", op, M=W * S, N=N, K=K, dtype="bf16", out_dtype="bf16", dist="int", world=W, rank=r,
                    shard_rows=S, chunks_per_shard=Q, order="ring" if op == "ag" else "rs_ring")
    d = si.draw(w)
    chunks, order = oracle.uniform_schedule(W, r, S, Q, w.order)
    cfg = {"timeout_ms": 1000, "bm": tile[0], "bn": tile[1], "bk": 64, "split_k": split}
    plan = csg.Plan(op, W * S, N, K, "bf16", "bf16", csg.Schedule.uniform(W, r, S, Q, w.order), cfg=cfg)
    if op == "ag":
        c, _ = run_ag(plan, chunks, d.A, d.B, "bf16", repeats=2)
        R = oracle.ag_gemm(d.A.device_array, d.B.device_array, chunks, order)
    else:
        c, _ = run_rs(plan, d.A, d.B, "bf16", repeats=2)
        R, _, _ = oracle.gemm_rs(d.A.device_array, d.B.device_array, chunks, order)
    assert np.array_equal(out_to_f64(c, "bf16"), bf16_rne_of_f64(R))
    plan.close()


@pytest.mark.parametrize("steps,split", [(1, 1), (2, 1), (3, 1), (5, 1), (8, 1), (9, 1), (5, 3), (7, 2), (12, 5)])
@pytest.mark.parametrize("op", ["ag", "rs"])
def test_fp32_pipeline_edges_bit_exact(steps, split, op):
    """The fp32 loop's stages hold two K steps of 16: whole and half last stages, slices that
    begin and end inside a stage, fewer stages than the ring."""
    W, r, S, N, K = 2, 1, 65, 64 + 4, 16 * steps
    print("fp32 loop", steps, split, op, flush=True)
    w = si.Workload(133, "loop", op, M=W * S, N=N, K=K, dtype="f32", out_dtype="f32", dist="int", world=W, rank=r,
                    shard_rows=S, chunks_per_shard=1, order="ring" if op == "ag" else "rs_ring")
    d = si.draw(w)
    chunks, order = oracle.uniform_schedule(W, r, S, 1, w.order)
    plan = csg.Plan(op, W * S, N, K, "f32", "f32", csg.Schedule.uniform(W, r, S, 1, w.order),
                    cfg={"timeout_ms": 1000, "split_k": split})
    if op == "ag":
        c, _ = run_ag(plan, chunks, d.A, d.B, "f32", repeats=2)
        R = oracle.ag_gemm(d.A.device_array, d.B.device_array, chunks, order)
    else:
        c, _ = run_rs(plan, d.A, d.B, "f32", repeats=2)
        R, _, _ = oracle.gemm_rs(d.A.device_array, d.B.device_array, chunks, order)
    assert np.array_equal(out_to_f64(c, "f32"), R)
    plan.close()


@pytest.mark.parametrize("split", [2, 3])
def test_wide_stores_of_split_tiles_hold_on_every_call(split):
    """fp32 output and partial sums leave as 16-byte stores, whose registers the next run's
    arithmetic reuses: forty calls, each bit for bit (a lost register showed in one call of
    ten)."""
    W, S, N, K = 2, 1280, 648, 512
    print("wide stores", split, flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(5)
    a = torch.randint(-2, 3, (W * S, K), generator=g, device="cuda:0").to(torch.bfloat16)
    b = torch.randint(-2, 3, (N, K), generator=g, device="cuda:0").to(torch.bfloat16)
    want = a.float() @ b.float().t()               # exact: every sum is below 2^24
    plan = csg.Plan("ag", W * S, N, K, "bf16", "f32", csg.Schedule.uniform(W, 0, S, 5, "ring"),
                    cfg={"split_k": split, "timeout_ms": 1000})
    st, cp = torch.cuda.Stream(), torch.cuda.Stream()
    land, c = a.clone(), torch.empty_like(want)
    for i in range(40):
        c.fill_(float("nan"))
        torch.cuda.synchronize()
        plan.ag_gemm(land, a, b, c, "overlap", st, cp)
        plan.check()
        torch.cuda.synchronize()
        assert torch.equal(c, want), i
    plan.close()
