"""GPU parity of default plans whose launch the library cuts into smaller tiles and
K-slices (launches that would leave most CUs idle): every tile that the library alone
chooses, with two, more and no slices, the choice itself checked where a plan reports it
(256 CUs). Integer inputs in {-2..2}: every sum is
below 2^24, so it is exact in fp32 whatever the order, and C must equal a plain fp32 product
(rounded once for bf16 output) bit for bit; the outgoing rows must equal C's."""
import numpy as np
import pytest

import paper_2601_20595_amd as csg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    # op, W, shard rows, q, N, K, out, cfg, the tile and slices it runs
    ("ag", 4, 1, 1, 132, 128, "bf16", {}, (128, 64, 1)),     # 4 rows, ragged last column tile
    ("ag", 2, 64, 2, 1792, 4096, "bf16", {}, (128, 64, 4)),
    ("ag", 4, 33, 3, 260, 1088, "f32", {}, (128, 64, 3)),    # 17 K steps, slices of unequal length
    ("ag", 2, 512, 4, 1796, 2048, "f32", {}, (128, 64, 1)),
    ("ag", 2, 1024, 4, 1792, 4096, "f32", {}, (128, 128, 1)),
    ("ag", 2, 1024, 4, 1792, 4096, "bf16", {}, (128, 128, 1)),
    ("ag", 2, 2048, 4, 1792, 4096, "bf16", {}, (256, 256, 2)),
    ("ag", 2, 1024, 4, 2052, 4096, "f32", {}, (256, 256, 3)),
    ("ag", 2, 300, 1, 1228, 2048, "bf16", {"copy_backend": "kernel", "copy_workgroups": 9}, (128, 64, 2)),
    # a copier in every slot
    ("ag", 2, 300, 1, 260, 640, "bf16", {"copy_backend": "kernel", "copy_workgroups": 249}, (256, 256, 1)),
    ("ag", 2, 300, 1, 260, 640, "bf16", {"copy_backend": "kernel", "copy_workgroups": 256}, (256, 256, 1)),
    ("ag", 2, 300, 2, 520, 640, "bf16", {"intra_order": 1, "tile_dispatch": 2}, (128, 64, 1)),
    ("rs", 2, 64, 2, 516, 2048, "bf16", {}, (128, 64, 4)),
    ("rs", 2, 640, 2, 1032, 512, "f32", {}, (128, 64, 1)),
    ("rs", 2, 1024, 4, 1792, 4096, "bf16", {}, (128, 128, 1)),
    ("rs", 2, 1024, 4, 1792, 4096, "f32", {}, (128, 128, 1)),
    ("rs", 2, 512, 4, 1284, 4096, "f32", {}, (128, 128, 2)),
    ("rs", 2, 640, 2, 772, 4096, "bf16", {}, (128, 128, 3)),
    ("rs", 2, 256, 1, 512, 1024, "bf16", {"copy_backend": "kernel"}, (128, 64, 1)),
    ("ar", 2, 256, 2, 516, 512, "bf16", {}, (128, 128, 1)),
    ("ar", 2, 256, 1, 260, 192, "f32", {}, (128, 128, 1)),
    ("grouped", 4, 0, 0, 264, 2048, "bf16", {}, (128, 64, 4)),
    ("grouped", 4, 0, 0, 1028, 256, "f32", {}, (128, 64, 1)),
    ("grouped", 4, 0, 0, 1792, 4096, "bf16", {}, (128, 128, 3)),
    ("grouped", 4, 0, 0, 1796, 4096, "f32", {}, (128, 128, 2)),
    ("noalloc", 8, 16, 1, 1792, 4096, "bf16", {}, None),
    ("noalloc", 2, 300, 3, 260, 1088, "f32", {}, None),
    ("noalloc", 2, 1024, 4, 1792, 4096, "f32", {}, None),
    ("noalloc", 2, 300, 1, 260, 640, "bf16", {"copy_workgroups": 256}, None),
]
F32_CASES = [
    ("ag", 2, 128, 2, 256, 2048, "f32", {}, (64, 64, 8)),
    ("ag", 2, 100, 2, 260, 528, "f32", {}, (64, 64, 3)),     # 33 K steps of 16 in three slices
    ("rs", 2, 100, 2, 260, 528, "f32", {}, (64, 64, 3)),
    ("ar", 2, 128, 2, 256, 2048, "f32", {}, (64, 64, 1)),    # the all-reduce splits no tile
    ("grouped", 4, 0, 0, 68, 1040, "f32", {}, (64, 64, 6)),
    ("noalloc", 2, 128, 2, 256, 2048, "f32", {}, None),
]


def _ints(shape, seed, dtype=torch.bfloat16):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return torch.randint(-2, 3, shape, generator=g, device=DEV).to(dtype)


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s-W%d-S%d-Q%d-N%d-K%d-%s-%s" % (
    c[:7] + ("_".join(sorted(c[7])) or "default",)))
def test_cut_launches_bit_exact(case):
    _run(case, "bf16")


@pytest.mark.parametrize("case", F32_CASES, ids=lambda c: "%s-W%d-S%d-Q%d-N%d-K%d" % c[:6])
def test_cut_fp32_launches_bit_exact(case):
    _run(case, "f32")


def _run(case, dtype):
    op, W, S, q, N, K, out, cfg, geometry = case
    print("geometry", dtype, case, flush=True)
    rank, ot = W - 1, torch.bfloat16 if out == "bf16" else torch.float32
    it = torch.bfloat16 if dtype == "bf16" else torch.float32
    groups = None
    if op == "grouped":
        counts = np.array([[70, 0, 5], [0, 3, 1], [130, 0, 0], [1, 2, 300]], dtype=np.int64)
        groups = counts.sum(axis=0).tolist()
        M, sched = int(counts.sum()), csg.Schedule.grouped(W, rank, counts)
    else:
        M, sched = W * S, csg.Schedule.uniform(W, rank, S, q, "rs_ring" if op in ("rs", "ar") else "ring")
    chunks, _ = sched.get()
    a = _ints((M, K), 1, it)
    b = _ints((len(groups), N, K) if groups else (N, K), 2, it)
    if groups:
        ref = torch.cat([a[lo:lo + n].float() @ b[e].float().t()
                         for e, (lo, n) in enumerate(zip(np.cumsum([0] + groups[:-1]).tolist(), groups)) if n])
    else:
        ref = a.float() @ b.float().t()
    c = torch.full((M, N), float("nan"), device=DEV, dtype=ot)
    st, cp = torch.cuda.Stream(), torch.cuda.Stream()
    plan = None if op == "noalloc" else csg.Plan(op, M, N, K, dtype, out, sched, group_rows=groups,
                                                 cfg=dict(cfg, timeout_ms=1000, trace=1))
    for _ in range(3):
        c.fill_(float("nan"))
        if op in ("ag", "grouped", "noalloc"):
            land = a.clone()
            for x in chunks:
                if not x[4]:
                    land[x[0]:x[1]] = float("nan")
            torch.cuda.synchronize()
            if op == "noalloc":
                csg.csg_ag_gemm_noalloc(sched, M, N, K, dtype, out, land, a, b, c, "overlap", cfg.get("copy_workgroups", 0), stream=st)
            else:
                (plan.ag_gemm if op == "ag" else plan.grouped_gemm)(land, a, b, c, "overlap", st, cp)
        else:
            sent = torch.zeros_like(c)
            if op == "ar":
                part = _ints((W - 1, S, N), 3).to(ot)
                part_land, reduced = torch.zeros_like(part), _ints((M, N), 4).to(ot)
                torch.cuda.synchronize()
                plan.gemm_ar(a, b, c, sent, part, part_land, reduced, "overlap", st, cp)
            else:
                torch.cuda.synchronize()
                plan.gemm_rs(a, b, c, sent, "overlap", st, cp)
        if plan:
            plan.check()
        torch.cuda.synchronize()
        if op == "ar":
            own = slice(rank * S, rank * S + S)
            want, want_sent = reduced.clone(), ref.to(ot, copy=True)
            want[own] = (ref[own] + part.float().sum(dim=0)).to(ot)
            want_sent[own] = want[own]
            assert torch.equal(c, want) and torch.equal(sent, want_sent)
            continue
        assert torch.equal(c, ref.to(ot))
        if op == "rs":
            assert all(torch.equal(sent[x[0]:x[1]], c[x[0]:x[1]]) for x in chunks if not x[4])
    if plan:
        bm, bn, split = geometry
        rows = groups if groups else [M]
        assert plan.info.n_units == sum(-(-r // bm) for r in rows) * -(-N // bn) * split
        assert set(plan.trace()["n_slices"].tolist()) == {split}
        plan.close()


def test_a_cut_plan_keeps_its_map_and_reports_its_own_tiles():
    W, S, N, K = 2, 300, 1228, 1024
    sched = csg.Schedule.uniform(W, 0, S, 2, "ring")
    host = csg.Plan("ag", W * S, N, K, "bf16", "bf16", sched, device=-1)
    plan = csg.Plan("ag", W * S, N, K, "bf16", "bf16", sched, cfg={"trace": 1, "timeout_ms": 1000})
    for x, y in zip(plan.get_map().values(), host.get_map().values()):
        assert np.array_equal(x, y)
    info = plan.info
    assert (info.bm, info.bn, info.n_tiles) == (256, 256, 15) and info.n_units > info.n_tiles
    a, b = _ints((W * S, K), 1), _ints((N, K), 2)
    c = torch.empty((W * S, N), device=DEV, dtype=torch.bfloat16)
    st, cp = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    plan.ag_gemm(a, a, b, c, "compute_only", st, cp)
    plan.check()
    tr = plan.trace()
    assert len(tr) == info.n_units and set(tr["raster"].tolist()) == set(range(info.n_tiles))
    plan.close()
