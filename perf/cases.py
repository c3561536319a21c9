"""The calls whose speed is watched, from the smallest to the largest, one per kind of use.

Every case is one call of the library as a program makes it, on a plan that the program
keeps, over simulated ranks of a tensor-, expert- or sequence-parallel layer. Shapes are
the FFN and attention slices of the 8B-like (hidden 4096, FFN 14336 / 8 = 1792) and
70B-like (hidden 8192, FFN 28672 / 8 = 3584) layers of the benchmark's workloads, the
tests' ragged shapes, and generic sizes between them.

A case's fields: op, dtype (input elements), out (output elements), world and rank,
shard (rows per rank), q (chunks per shard), order, n, k, and cfg, the plan
configuration as JSON text ("" = the library's default plan). Grouped GEMMs have tokens,
experts and topk instead of shards; attention has heads, kv_heads and rows (queries).
"""
import json
import math

import numpy as np
import torch

import paper_2601_20595_amd as csg

DEV = "cuda:0"
HEAD_DIM = 128
TORCH = {"bf16": torch.bfloat16, "f32": torch.float32}
SIZE = {"bf16": 2, "f32": 4}
ZIPF = 1.2  # skew of the routing over experts
TILE_128 = '{"bm": 128, "bn": 256, "bk": 64, "tile_dispatch": 2}'
FINE_PLAN = ('{"bm": 128, "bn": 256, "bk": 64, "tile_dispatch": 2, "tail_split": 4, "tail_chunks": 12, '
             '"tail_taper": 1, "copy_split": 2}')
KERNEL_COPIES = '{"copy_backend": "kernel", "copy_workgroups": 64}'


def _gemm(name, op, dtype, out, world, rank, shard, q, order, n, k, cfg=""):
    return dict(name=name, op=op, dtype=dtype, out=out, world=world, rank=rank, shard=shard, q=q, order=order, n=n,
                k=k, cfg=cfg)


def _grouped(name, tokens, experts, topk, world, rank, n, k, out="bf16", cfg=""):
    return dict(name=name, op="grouped", dtype="bf16", out=out, world=world, rank=rank, tokens=tokens,
                experts=experts, topk=topk, n=n, k=k, cfg=cfg)


def _attn(name, rows, heads, kv_heads, world, rank, shard, q, order="ring"):
    return dict(name=name, op="attn", dtype="bf16", out="bf16", world=world, rank=rank, rows=rows, heads=heads,
                kv_heads=kv_heads, shard=shard, q=q, order=order, cfg="")


def listed():
    return [
        # the smallest call: two ranks, fp32; launch, copy and flag latency
        _gemm("ag_f32_256", "ag", "f32", "f32", 2, 0, 128, 2, "permutation", 256, 256),
        # a decode step: 16 tokens per rank gathered for the up-projection, from a serving
        # loop that allocates nothing
        _gemm("noalloc_decode", "noalloc", "bf16", "bf16", 8, 0, 16, 1, "ring", 1792, 4096),
        # a ragged prefill on four ranks, chunks that straddle tiles, fp32 output
        _gemm("ag_ragged", "ag", "bf16", "f32", 4, 3, 300, 2, "ring", 1228, 2048),
        # a prompt's up-projection on the 8B-like layer, default plan
        _gemm("ag_8b", "ag", "bf16", "bf16", 8, 0, 1024, 4, "ring", 1792, 4096),
        # long prefill on the 70B-like layer with fine chunks, the plan tuned for it
        _gemm("ag_70b_fine", "ag", "bf16", "bf16", 8, 0, 2048, 16, "permutation", 3584, 8192, FINE_PLAN),
        # the row-parallel down-projection with reduce-scatter, default plan
        _gemm("rs_8b", "rs", "bf16", "bf16", 8, 0, 1024, 4, "rs_ring", 4096, 1792),
        # the same operation in fp32 at an ordinary size
        _gemm("rs_f32", "rs", "f32", "f32", 4, 1, 512, 2, "rs_ring", 1024, 1024),
        # the down-projection with all-reduce
        _gemm("ar_8b", "ar", "bf16", "bf16", 8, 0, 1024, 4, "rs_ring", 4096, 1792),
        # mixture of experts: a large batch routed to eight experts
        _grouped("moe_8b", 16384, 8, 2, 8, 0, 1792, 4096),
        # mixture of experts: a small batch, a few dozen ragged rows per expert
        _grouped("moe_decode", 256, 8, 2, 8, 3, 1792, 4096),
        # sequence-parallel attention over 32k keys
        _attn("attn_32k", 4096, 32, 8, 8, 0, 4096, 2),
        # a short ragged prompt of a few hundred rows per rank
        _attn("attn_short", 500, 32, 8, 4, 2, 512, 2),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        c = _draw(rng)
        # no costlier than the largest listed cases
        if work(c)["flops"] <= 9e11 and work(c)["bytes"] <= 6e8:
            return c


def _draw(rng):
    op = rng.choice(["ag", "ag", "ag", "noalloc", "rs", "rs", "ar", "grouped", "grouped", "attn", "attn"])
    world = rng.choice([2, 4, 8])
    rank = rng.randrange(world)
    if op == "attn":
        kv = rng.choice([1, 2, 4, 8])
        c = _attn("", _log(rng, 64, 4096), kv * rng.choice([1, 2, 4]), kv, world, rank, 0, rng.choice([1, 2, 4]))
        c["shard"] = 64 * c["q"] * max(1, _log(rng, 128, 4096) // (64 * c["q"]))
        c["order"] = rng.choice(["ring", "swizzle1d"])
    elif op == "grouped":
        c = _grouped("", _log(rng, 64, 16384), rng.choice([4, 8, 16]), rng.choice([1, 2]), world, rank,
                     4 * _log(rng, 64, 1024), 64 * _log(rng, 8, 96), rng.choice(["bf16", "bf16", "f32"]))
        c["tokens"] = world * max(1, c["tokens"] // world)
        if c["out"] == "bf16" and rng.random() < 0.2:
            c["cfg"] = rng.choice([TILE_128, KERNEL_COPIES])
    else:
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
        out = rng.choice(["bf16", "bf16", "f32"]) if dtype == "bf16" else "f32"
        q = rng.choice([1, 2, 4])
        rows = _log(rng, 64, 16384 if dtype == "bf16" else 4096)
        shard = q * max(1, rows // (world * q))
        k = 64 * _log(rng, 4, 128) if dtype == "bf16" else 16 * _log(rng, 8, 128)
        n = 4 * _log(rng, 32, 1024)
        order = "rs_ring" if op in ("rs", "ar") else rng.choice(["ring", "swizzle1d", "permutation"])
        if op == "ar":  # shards of whole tile rows
            tile = 256 if dtype == "bf16" else 64
            shard = tile * max(1, shard // tile)
        cfg = ""
        if op == "ag" and dtype == "bf16" and out == "bf16" and rng.random() < 0.3:
            cfg = rng.choice([TILE_128, KERNEL_COPIES])
        c = _gemm("", op, dtype, out, world, rank, shard, q, order, n, k, cfg)
    del c["name"]
    return c


# ---- what a program has in hand before the call ------------------------------------
_streams = []


def _stream_pair():
    """The program's compute and copy streams."""
    if not _streams:
        _streams.extend((torch.cuda.Stream(device=DEV), torch.cuda.Stream(device=DEV)))
    return _streams


def _gen(seed, stream):
    return torch.Generator(device=DEV).manual_seed((seed % (1 << 30)) * 16 + stream)


def _normal(seed, stream, shape, scale, dtype):
    x = torch.randn(shape, generator=_gen(seed, stream), device=DEV, dtype=torch.float32)
    return x.mul_(scale).to(TORCH[dtype])


def _routing(case, seed):
    """Rows per (source rank, expert): every token picks topk experts by Gumbel top-k
    over Zipf weights."""
    g = np.random.default_rng([seed % (1 << 30), 4])
    logw = -ZIPF * np.log(np.arange(1, case["experts"] + 1, dtype=np.float64))
    keys = logw[None, :] + g.gumbel(size=(case["tokens"], case["experts"]))
    top = np.argsort(-keys, axis=1)[:, :case["topk"]]
    src = np.arange(case["tokens"]) // (case["tokens"] // case["world"])
    counts = np.zeros((case["world"], case["experts"]), dtype=np.int64)
    np.add.at(counts, (np.repeat(src, case["topk"]), top.reshape(-1)), 1)
    return counts


def _rows(case):
    return case["tokens"] * case["topk"] if case["op"] == "grouped" else case["world"] * case["shard"]


def _schedule(case, seed):
    if case["op"] == "grouped":
        return csg.Schedule.grouped(case["world"], case["rank"], _routing(case, seed))
    perm = None
    if case["order"] == "permutation":
        perm = np.random.default_rng([seed % (1 << 30), 2]).permutation((case["world"] - 1) * case["q"])
    return csg.Schedule.uniform(case["world"], case["rank"], case["shard"], case["q"], case["order"], perm)


def _inputs(case, seed):
    """The call's input tensors, by name."""
    op = case["op"]
    if op == "attn":
        keys = (case["world"] * case["shard"], case["kv_heads"], HEAD_DIM)
        return {"q": _normal(seed, 0, (case["rows"], case["heads"], HEAD_DIM), 1.0, "bf16"),
                "k": _normal(seed, 1, keys, 1.0, "bf16"), "v": _normal(seed, 2, keys, 1.0, "bf16")}
    m, n, k = _rows(case), case["n"], case["k"]
    d = {"a": _normal(seed, 0, (m, k), 0.02, case["dtype"])}
    if op == "grouped":
        d["b"] = _normal(seed, 1, (case["experts"], n, k), 0.02, case["dtype"])
    else:
        d["b"] = _normal(seed, 1, (n, k), 0.02, case["dtype"])
    if op == "ar":
        # partial sums of the other ranks and the reduced rows that their owners send
        s = 0.02 * 0.02 * math.sqrt(k)
        d["partials"] = _normal(seed, 5, (case["world"] - 1, case["shard"], n), s, case["out"])
        d["reduced"] = _normal(seed, 6, (m, n), s * math.sqrt(case["world"]), case["out"])
    return d


def _zero_remote(t, chunks):
    for c in chunks:
        if not c[4]:
            t[c[0]:c[1]].zero_()


def prepare(case, seed):
    op = case["op"]
    sched = _schedule(case, seed)
    chunks, _ = sched.get()
    d = _inputs(case, seed)
    s = {"case": case, "sched": sched, "streams": _stream_pair(), **d}
    cfg = json.loads(case["cfg"]) if case["cfg"] else None
    if op == "attn":
        s["plan"] = csg.AttnPlan(case["heads"], case["kv_heads"], HEAD_DIM, case["rows"], sched, cfg=cfg)
        s["k_land"], s["v_land"] = d["k"].clone(), d["v"].clone()
        _zero_remote(s["k_land"], chunks)
        _zero_remote(s["v_land"], chunks)
        s["o"] = torch.empty_like(d["q"])
        s["lse"] = torch.empty((case["heads"], case["rows"]), dtype=torch.float32, device=DEV)
        return s
    m, n, k = _rows(case), case["n"], case["k"]
    if op != "noalloc":
        groups = _routing(case, seed).sum(axis=0).tolist() if op == "grouped" else None
        s["plan"] = csg.Plan(op, m, n, k, case["dtype"], case["out"], sched, group_rows=groups, cfg=cfg)
    s["c"] = torch.empty((m, n), dtype=TORCH[case["out"]], device=DEV)
    if op in ("ag", "noalloc", "grouped"):
        s["landing"] = d["a"].clone()
        _zero_remote(s["landing"], chunks)
    else:
        s["outgoing"] = torch.zeros((m, n), dtype=TORCH[case["out"]], device=DEV)
    if op == "ar":
        s["partials_land"] = torch.zeros_like(d["partials"])
    return s


def run(s):
    case = s["case"]
    compute, copy = s["streams"]
    op = case["op"]
    if op == "attn":
        s["plan"].ring_attn(s["q"], s["k_land"], s["v_land"], s["k"], s["v"], s["o"], s["lse"], "overlap", compute, copy)
        return {"o": s["o"], "lse": s["lse"], "k": s["k_land"], "v": s["v_land"]}
    if op == "noalloc":
        csg.csg_ag_gemm_noalloc(s["sched"], _rows(case), case["n"], case["k"], case["dtype"], case["out"], s["landing"],
                                s["a"], s["b"], s["c"], "overlap", 0, 0, compute)
        return {"c": s["c"], "landing": s["landing"]}
    p = s["plan"]
    if op in ("ag", "grouped"):
        call = p.ag_gemm if op == "ag" else p.grouped_gemm
        call(s["landing"], s["a"], s["b"], s["c"], "overlap", compute, copy)
        return {"c": s["c"], "landing": s["landing"]}
    # the copies out end after the call: what follows on the stream waits for them
    if op == "rs":
        p.gemm_rs(s["a"], s["b"], s["c"], s["outgoing"], "overlap", compute, copy)
    else:
        p.gemm_ar(s["a"], s["b"], s["c"], s["outgoing"], s["partials"], s["partials_land"], s["reduced"], "overlap",
                  compute, copy)
    p.join(compute)
    return {"c": s["c"], "outgoing": s["outgoing"]}


# ---- what a pass cannot do without ---------------------------------------------------
def work(case):
    w, op = case["world"], case["op"]
    ib, ob = SIZE[case["dtype"]], SIZE[case["out"]]
    remote = (w - 1) / w
    if op == "attn":
        q, kv = case["rows"] * case["heads"] * HEAD_DIM, w * case["shard"] * case["kv_heads"] * HEAD_DIM
        return {"bytes": 2 * (2 * q + 2 * kv + 2 * kv * remote) + 4 * case["rows"] * case["heads"],
                "flops": 4.0 * case["rows"] * w * case["shard"] * case["heads"] * HEAD_DIM}
    m, n, k = _rows(case), case["n"], case["k"]
    experts = case.get("experts", 1)
    b = m * k * ib + experts * n * k * ib + m * n * ob
    if op in ("ag", "noalloc", "grouped"):
        b += m * k * ib * remote                      # the landed rows
    else:
        b += m * n * ob * (remote if op == "rs" else 1)  # the rows sent
    if op == "ar":
        b += 2 * (w - 1) * case["shard"] * n * ob + m * n * ob * remote  # partials in and landed, reduced rows in
    return {"bytes": b, "flops": 2.0 * m * n * k}


# bf16 results: rounding to bf16 leaves 1.7e-3 of the norm against 64 bits, one unit in
# the last place at most where the sum's order moves a result across a rounding boundary
# (attention's weights are bf16 too). fp32 results: 2e-7 to 6e-7 seen for sums of 256 to
# 2048 products, which grow with the square root of their number.
def tolerance(case):
    if case["out"] == "bf16":
        return {"rel": 7e-3, "max": 4e-2}
    return {"rel": 5e-6, "max": 5e-5}


# ---- the same results in 64 bits -----------------------------------------------------
def exact(case, seed):
    op = case["op"]
    d = {x: t.double() for x, t in _inputs(case, seed).items()}
    chunks, _ = _schedule(case, seed).get()
    if op == "attn":
        group = case["heads"] // case["kv_heads"]
        o = torch.empty_like(d["q"])
        lse = torch.empty((case["heads"], case["rows"]), dtype=torch.float64, device=DEV)
        for h in range(case["heads"]):
            sc = (d["q"][:, h].contiguous() @ d["k"][:, h // group].t().contiguous()).mul_(1.0 / math.sqrt(HEAD_DIM))
            top = sc.amax(dim=1, keepdim=True)
            sc.sub_(top).exp_()
            total = sc.sum(dim=1, keepdim=True)
            o[:, h] = (sc @ d["v"][:, h // group].contiguous()).div_(total)
            lse[h] = (total.log() + top)[:, 0]
        return {"o": o, "lse": lse, "k": d["k"], "v": d["v"]}
    if op == "grouped":
        c = torch.empty((_rows(case), case["n"]), dtype=torch.float64, device=DEV)
        for x in chunks:
            c[x[0]:x[1]] = d["a"][x[0]:x[1]] @ d["b"][x[3]].t()
    else:
        c = d["a"] @ d["b"].t()
    if op in ("ag", "noalloc", "grouped"):
        return {"c": c, "landing": d["a"]}
    out = c.clone()
    if op == "rs":
        own = [x for x in chunks if x[4]]
        for x in own:
            out[x[0]:x[1]] = 0.0
        return {"c": c, "outgoing": out}
    lo = case["rank"] * case["shard"]
    hi = lo + case["shard"]
    own = c[lo:hi] + d["partials"].sum(dim=0)
    c = d["reduced"].clone()
    c[lo:hi] = own
    out[lo:hi] = own
    return {"c": c, "outgoing": out}
