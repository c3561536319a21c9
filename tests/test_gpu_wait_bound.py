"""The bound on a unit's wait for several chunks: chunks that land one after another, each
within timeout_ms of the one before, are waited for however long they take in all, and a
chunk that stays away longer than that after the last one ends the call with its name."""
import pytest

import paper_2601_20595_amd as csg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _call(cfg, delays_us, S=16, K=128):
    """One overlap call of six ranks' rows in one row tile (five remote chunks)."""
    W, N = 6, 128
    dtype = "f32" if K == 64 else "bf16"
    t = torch.float32 if K == 64 else torch.bfloat16
    sched = csg.Schedule.uniform(W, 0, S, 1, "ring")
    plan = csg.Plan("ag", W * S, N, K, dtype, dtype, sched, cfg=dict(cfg, timeout_ms=200))
    plan.set_copy_delays(delays_us)
    g = torch.Generator(device=DEV).manual_seed(3)
    a = torch.randint(-2, 3, (W * S, K), generator=g, device=DEV).to(t)
    b = torch.randint(-2, 3, (N, K), generator=g, device=DEV).to(t)
    land, c = a.clone(), torch.empty((W * S, N), device=DEV, dtype=t)
    land[S:] = float("nan")
    st, cp = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    plan.ag_gemm(land, a, b, c, "overlap", st, cp)
    try:
        plan.check()
        return c, (a.float() @ b.float().t()).to(t), plan
    finally:
        torch.cuda.synchronize()


@pytest.mark.parametrize("cfg,S,K", [({}, 16, 128), ({"tile_dispatch": 2}, 16, 128), ({}, 8, 64)],
                         ids=["relay", "static", "f32"])
def test_chunks_that_land_one_after_another_are_waited_for(cfg, S, K):
    print("wait bound", cfg, S, K, flush=True)
    c, want, plan = _call(cfg, [120000.0] * 5, S, K)    # the last lands after 600 ms
    assert torch.equal(c, want)
    plan.close()


@pytest.mark.parametrize("cfg", [{}, {"tile_dispatch": 2}], ids=["relay", "static"])
def test_a_chunk_that_stays_away_ends_the_call(cfg):
    print("wait bound, late", cfg, flush=True)
    with pytest.raises(csg.CsgError) as e:
        _call(cfg, [120000.0, 120000.0, 500000.0, 0.0, 0.0])
    assert e.value.status == csg.CSG_ERR_TIMEOUT
    _, order = csg.Schedule.uniform(6, 0, 16, 1, "ring").get()
    assert e.value.diag.chunk in [x for x in order if x != 0][2:]
