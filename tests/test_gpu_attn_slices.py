"""GPU parity of ring attention whose units are cut along the keys (few query rows and
heads): slices of unequal length, slices that begin inside a chunk, chunks no slice of a
unit reads, rows whose largest score lies in one slice only, calls in a row on one plan.
Against plain attention in 64 bits; bf16 weights bound the error at 2e-2 of the result."""
import math
import time

import numpy as np
import pytest

import paper_2601_20595_amd as csg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    # rows, heads, kv heads, chunk rows (multiples of 64), local chunks, slices
    (100, 2, 1, [64] * 13, {0, 1}, 2),                 # 13 blocks: slices of 6 and 7
    (1, 4, 2, [64 * 24], {0}, 4),                      # one chunk: every slice inside it
    (300, 3, 3, [64, 448, 128, 1024, 64, 320], {2}, 5),  # uneven chunks
    (70, 3, 3, [64, 448, 128, 1024, 64, 1344], {2}, 8),
    (128, 1, 1, [64 * 11], set(), 1),                  # 11 blocks: not cut
    (4100, 16, 4, [512, 512, 256], {1}, 1),            # more units than slots: not cut
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "q%d-h%d-kv%d-n%d" % (c[0], c[1], c[2], len(c[3])))
@pytest.mark.parametrize("spread", [1.0, 8.0])
def test_sliced_attention_parity(case, spread):
    rows, H, Hkv, sizes, local, slices = case
    print("attention slices", case, spread, flush=True)
    ends = np.cumsum(sizes).tolist()
    chunks = [(e - s, e, 0 if i in local else 1 + i, 0, int(i in local)) for i, (e, s) in enumerate(zip(ends, sizes))]
    order = sorted(range(len(sizes)), key=lambda i: (i not in local, -i))
    plan = csg.AttnPlan(H, Hkv, 128, rows, csg.Schedule.create(chunks, order), cfg={"timeout_ms": 1000})
    assert plan.info.n_units == (rows + 127) // 128 * H * slices
    g = torch.Generator(device=DEV).manual_seed(7)
    S = ends[-1]
    q = torch.randn((rows, H, 128), generator=g, device=DEV).to(torch.bfloat16)
    # the keys' scale grows along the sequence: with a spread of 8 the last keys hold the maxima
    k = (torch.randn((S, Hkv, 128), generator=g, device=DEV) *
         torch.linspace(1.0 / spread, 1.0, S, device=DEV)[:, None, None]).to(torch.bfloat16)
    v = torch.randn((S, Hkv, 128), generator=g, device=DEV).to(torch.bfloat16)
    o, lse = torch.empty_like(q), torch.empty((H, rows), device=DEV)
    st, cp = torch.cuda.Stream(), torch.cuda.Stream()
    first = None
    for _ in range(3):
        kl, vl = k.clone(), v.clone()
        for c in chunks:
            if not c[4]:
                kl[c[0]:c[1]] = float("nan")
                vl[c[0]:c[1]] = float("nan")
        o.fill_(float("nan"))
        torch.cuda.synchronize()
        plan.ring_attn(q, kl, vl, k, v, o, lse, "overlap", st, cp)
        plan.check()
        torch.cuda.synchronize()
        first = o.clone() if first is None else first
        assert torch.equal(o, first)               # merged in slice order: the same bits every time
    for h in range(H):
        s = (q[:, h].double() @ k[:, h * Hkv // H].double().t()) / math.sqrt(128)
        want = torch.softmax(s, dim=1) @ v[:, h * Hkv // H].double()
        err = (o[:, h].double() - want).abs().max() / want.square().mean().sqrt()
        assert err <= 2e-2 * max(1.0, float(want.abs().max() / want.square().mean().sqrt())), (h, float(err))
        assert (lse[h].double() - torch.logsumexp(s, dim=1)).abs().max() <= 2e-2
    plan.close()


def test_slices_of_keys_that_score_minus_infinity_count_for_nothing():
    """Keys from the third slice on score -inf for every query: their slices have no finite
    maximum, and the result is that of the other keys."""
    rows, H, sizes = 128, 2, [64 * 12, 64 * 36]
    print("attention slices, -inf scores", flush=True)
    chunks = [(0, sizes[0], 0, 0, 1), (sizes[0], sum(sizes), 1, 0, 0)]
    plan = csg.AttnPlan(H, 1, 128, rows, csg.Schedule.create(chunks, [0, 1]), cfg={"timeout_ms": 1000})
    assert plan.info.n_units == 8 * H                     # eight slices of six blocks
    g = torch.Generator(device=DEV).manual_seed(9)
    q = torch.randn((rows, H, 128), generator=g, device=DEV).to(torch.bfloat16)
    q[:, :, 0] = q[:, :, 0].abs() + 0.5
    k = torch.randn((sum(sizes), 1, 128), generator=g, device=DEV).to(torch.bfloat16)
    v = torch.randn((sum(sizes), 1, 128), generator=g, device=DEV).to(torch.bfloat16)
    k[sizes[0]:, :, 0] = float("-inf")
    o, lse = torch.empty_like(q), torch.empty((H, rows), device=DEV)
    st, cp = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    plan.ring_attn(q, k.clone(), v.clone(), k, v, o, lse, "overlap", st, cp)
    plan.check()
    torch.cuda.synchronize()
    n = sizes[0]
    for h in range(H):
        s = (q[:, h].double() @ k[:n, 0].double().t()) / math.sqrt(128)
        want = torch.softmax(s, dim=1) @ v[:n, 0].double()
        scale = float(want.square().mean().sqrt())
        assert (o[:, h].double() - want).abs().max() <= 2e-2 * max(scale, float(want.abs().max()))
        assert (lse[h].double() - torch.logsumexp(s, dim=1)).abs().max() <= 2e-2
    plan.close()


SAME = [
    # rows, heads, kv heads, chunk rows, local chunks, arrival order
    (500, 32, 8, [256] * 8, {4, 5}, [4, 5, 6, 7, 0, 1, 2, 3]),   # four slices
    (300, 3, 3, [64, 448, 128, 1024, 64, 320], set(), [3, 0, 5, 1, 4, 2]),  # five; the first chunk arrives too
    (64, 2, 1, [64 * 12], {0}, [0]),                             # two slices of one chunk
]


@pytest.mark.parametrize("case", SAME, ids=lambda c: "q%d-h%d-kv%d-n%d" % (c[0], c[1], c[2], len(c[3])))
def test_slices_weigh_the_keys_as_the_uncut_kernel_does(case):
    """The same plan cut and uncut (num_workgroups named). Both round the same weights to
    bf16, so only the order of the fp32 sums differs: n keys in sums of fewer than n terms
    keep a relative error below n 2^-24 (about 1e-4 here; a few 1e-7 as errors average),
    which moves few results across a bf16 boundary and none further than to its
    neighbour."""
    rows, H, Hkv, sizes, local, order = case
    print("attention slices, cut and uncut", case, flush=True)
    ends = np.cumsum(sizes).tolist()
    S = ends[-1]
    chunks = [(e - s, e, 0 if i in local else 1 + i, 0, int(i in local)) for i, (e, s) in enumerate(zip(ends, sizes))]
    g = torch.Generator(device=DEV).manual_seed(11)
    q = torch.randn((rows, H, 128), generator=g, device=DEV).to(torch.bfloat16)
    k = torch.randn((S, Hkv, 128), generator=g, device=DEV).to(torch.bfloat16)
    v = torch.randn((S, Hkv, 128), generator=g, device=DEV).to(torch.bfloat16)
    st, cp = torch.cuda.Stream(), torch.cuda.Stream()
    out, units = [], []
    for cfg in ({"timeout_ms": 1000}, {"timeout_ms": 1000, "num_workgroups": 256}):
        plan = csg.AttnPlan(H, Hkv, 128, rows, csg.Schedule.create(chunks, order), cfg=cfg)
        o, lse = torch.empty_like(q), torch.empty((H, rows), device=DEV)
        kl, vl = k.clone(), v.clone()
        for c in chunks:
            if not c[4]:
                kl[c[0]:c[1]] = float("nan")
                vl[c[0]:c[1]] = float("nan")
        torch.cuda.synchronize()
        plan.ring_attn(q, kl, vl, k, v, o, lse, "overlap", st, cp)
        plan.check()
        torch.cuda.synchronize()
        out.append((o, lse))
        units.append(plan.info.n_units)
        plan.close()
    whole = (rows + 127) // 128 * H
    assert units[1] == whole and units[0] > whole          # the first plan is cut
    (o, lse), (uo, ulse) = out
    assert float((lse - ulse).abs().max()) <= S * 2.0 ** -24
    differ = (o != uo)
    print("differ", float(differ.float().mean()), "rel", float((o.double() - uo.double()).norm() / uo.double().norm()),
          "lse", float((lse - ulse).abs().max()), flush=True)
    # a sum's error of e moves it across a boundary with a chance of about e / 2^-9: 1e-3
    # of the results for 2e-6, ten times as many where terms of either sign cancel
    assert float(differ.float().mean()) <= 1e-2
    rms = float(uo.double().square().mean().sqrt())
    assert float(((o.double() - uo.double()).abs() / uo.double().abs().clamp(min=rms)).max()) <= 2.0 ** -7


@pytest.mark.parametrize("rows,num_workgroups", [(128, 0), (128, 64), (9000, 0)], ids=["cut", "uncut", "uncut-rows"])
@pytest.mark.parametrize("first", [64, 64 * 12], ids=["block", "chunk"])
def test_first_keys_that_score_minus_infinity_count_for_nothing(rows, num_workgroups, first):
    """The first keys to arrive score -inf for every query, alone and with the unit cut or
    not: the result is that of the other keys, and does not depend on how a call is cut."""
    H, sizes = 4, [64 * 24, first]
    print("attention, -inf first", rows, num_workgroups, first, flush=True)
    chunks = [(0, sizes[0], 0, 0, 1), (sizes[0], sum(sizes), 1, 0, 0)]
    plan = csg.AttnPlan(H, 1, 128, rows, csg.Schedule.create(chunks, [1, 0]),
                        cfg={"timeout_ms": 1000, "num_workgroups": num_workgroups})
    assert (plan.info.n_units == (rows + 127) // 128 * H) == (num_workgroups != 0 or rows != 128)
    g = torch.Generator(device=DEV).manual_seed(13)
    q = torch.randn((rows, H, 128), generator=g, device=DEV).to(torch.bfloat16)
    q[:, :, 0] = q[:, :, 0].abs() + 0.5
    k = torch.randn((sum(sizes), 1, 128), generator=g, device=DEV).to(torch.bfloat16)
    v = torch.randn((sum(sizes), 1, 128), generator=g, device=DEV).to(torch.bfloat16)
    k[sizes[0]:, :, 0] = float("-inf")
    o, lse = torch.empty_like(q), torch.empty((H, rows), device=DEV)
    st, cp = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    plan.ring_attn(q, k.clone(), v.clone(), k, v, o, lse, "overlap", st, cp)
    plan.check()
    torch.cuda.synchronize()
    n = sizes[0]
    for h in range(H):
        s = (q[:, h].double() @ k[:n, 0].double().t()) / math.sqrt(128)
        want = torch.softmax(s, dim=1) @ v[:n, 0].double()
        scale = float(want.square().mean().sqrt())
        assert (o[:, h].double() - want).abs().max() <= 2e-2 * max(scale, float(want.abs().max()))
        assert (lse[h].double() - torch.logsumexp(s, dim=1)).abs().max() <= 2e-2
    plan.close()


def test_slices_release_a_chunk_before_the_kernel_ends():
    """The first chunk is one block of two million keys, which eight slices walk for
    milliseconds: the next call's copy into its rows has to go ahead meanwhile, so two
    calls return (their copies complete) long before the first kernel ends."""
    sizes = [64, 64 * 32767]
    print("attention slices, early release", flush=True)
    chunks = [(0, 64, 1, 0, 0), (64, sum(sizes), 0, 0, 1)]
    plan = csg.AttnPlan(1, 1, 128, 128, csg.Schedule.create(chunks, [0, 1]), cfg={"timeout_ms": 1000})
    assert plan.info.n_units == 8
    g = torch.Generator(device=DEV).manual_seed(15)
    q = torch.randn((128, 1, 128), generator=g, device=DEV).to(torch.bfloat16)
    k = torch.randn((sum(sizes), 1, 128), generator=g, device=DEV).to(torch.bfloat16)
    v = torch.randn((sum(sizes), 1, 128), generator=g, device=DEV).to(torch.bfloat16)
    kl, vl = k.clone(), v.clone()
    o, lse = torch.empty_like(q), torch.empty((1, 128), device=DEV)
    st, cp = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    plan.ring_attn(q, kl, vl, k, v, o, lse, "overlap", st, cp)   # loads the kernel
    plan.check()
    torch.cuda.synchronize()
    first, kernel_ms = o.clone(), float(plan.kernel_times(1)[0])
    assert kernel_ms > 1.0
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    plan.ring_attn(q, kl, vl, k, v, o, lse, "overlap", st, cp)
    plan.ring_attn(q, kl, vl, k, v, o, lse, "overlap", st, cp)
    assert (time.perf_counter() - t0) * 1e3 < 0.5 * kernel_ms
    plan.check()
    torch.cuda.synchronize()
    assert torch.equal(o, first)
    plan.close()


@pytest.mark.parametrize("num_workgroups", [1, 24, 63, 64, 71, 72, 100, 504, 512])
def test_units_of_a_named_grid_are_spread_over_the_dies(num_workgroups):
    """64 units on grids of fewer, as many and more workgroups: the same bits, and a grid
    larger than the units is no slower than one of as many (the units of a 512-workgroup
    grid once ran on one die: 1.4 times the time)."""
    rows, H, S = 100, 64, 4096
    print("attention, named grid", num_workgroups, flush=True)
    g = torch.Generator(device=DEV).manual_seed(17)
    q = torch.randn((rows, H, 128), generator=g, device=DEV).to(torch.bfloat16)
    k = torch.randn((S, H, 128), generator=g, device=DEV).to(torch.bfloat16)
    v = torch.randn((S, H, 128), generator=g, device=DEV).to(torch.bfloat16)
    st, cp = torch.cuda.Stream(), torch.cuda.Stream()
    out, ms = [], []
    for n in (64, num_workgroups):
        plan = csg.AttnPlan(H, H, 128, rows, csg.Schedule.create([(0, S, 0, 0, 1)], [0]),
                            cfg={"timeout_ms": 1000, "num_workgroups": n})
        assert plan.info.n_units == 64
        o, lse = torch.full_like(q, float("nan")), torch.empty((H, rows), device=DEV)
        torch.cuda.synchronize()
        for _ in range(30):
            plan.ring_attn(q, k, v, k, v, o, lse, "compute_only", st, cp)
        plan.check()
        torch.cuda.synchronize()
        out.append((o, lse))
        ms.append(float(np.median(plan.kernel_times(20))))
        plan.close()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    print("ms", ms, flush=True)
    if num_workgroups >= 64:
        assert ms[1] <= 1.3 * ms[0]


@pytest.mark.parametrize("case,bound", [((1230, 32, 8, 640), 1.4), ((640, 32, 8, 1280), 1.8)], ids=["uncut", "cut"])
def test_waiting_units_do_not_hold_up_the_copies_they_wait_for(case, bound):
    """Calls in a row on one landing buffer, half of the keys copied. Every unit reaches the
    remote half at once; when all of them polled the copies' completion values, which lie in
    host memory, the polls slowed the copies: kernels of 80 and 99 us where compute-only
    ones took 55 and 46. They take 37 of 31 and 53 of 36 now (the cut units' remote slices
    have no local half to hide their copy behind)."""
    rows, H, Hkv, S = case
    print("attention, waiting units", case, flush=True)
    g = torch.Generator(device=DEV).manual_seed(19)
    q = torch.randn((rows, H, 128), generator=g, device=DEV).to(torch.bfloat16)
    k = torch.randn((S, Hkv, 128), generator=g, device=DEV).to(torch.bfloat16)
    v = torch.randn((S, Hkv, 128), generator=g, device=DEV).to(torch.bfloat16)
    kl, vl = k.clone(), v.clone()
    o, lse = torch.empty_like(q), torch.empty((H, rows), device=DEV)
    st, cp = torch.cuda.Stream(), torch.cuda.Stream()
    plan = csg.AttnPlan(H, Hkv, 128, rows, csg.Schedule.uniform(2, 1, S // 2, 1, "ring"), cfg={"timeout_ms": 1000})
    torch.cuda.synchronize()
    us = {}
    for mode in ("compute_only", "overlap"):
        for _ in range(60):
            plan.ring_attn(q, kl, vl, k, v, o, lse, mode, st, cp)
        plan.check()
        torch.cuda.synchronize()
        us[mode] = float(np.median(plan.kernel_times(40))) * 1e3
    print("us", us, flush=True)
    plan.close()
    assert us["overlap"] <= bound * us["compute_only"]
