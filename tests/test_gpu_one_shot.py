"""GPU parity of launches in which every work unit has a workgroup of its own: units dealt
statically, completion values relayed by one workgroup where slots are left, waits and
counts one chunk per lane (so more than 64 chunks per tile take several rounds, more than
512 remote chunks several per relay thread). Integer inputs: bit for bit."""
import numpy as np
import pytest

import oracle
import paper_2601_20595_amd as csg
import seeded_inputs as si

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from gpu_util import bf16_rne_of_f64, out_to_f64, run_ag, run_rs

CASES = [
    # op, W, S, Q, N, K, dtype, cfg, workgroups beside those of the units
    ("ag", 2, 700, 700, 260, 64, "bf16", {}, 8),      # 1-row chunks: 256 per tile, 700 relayed
    ("ag", 2, 100, 50, 64, 128, "f32", {}, 8),        # lines straddle chunks
    ("ag", 8, 2, 1, 516, 192, "bf16", {}, 8),         # 16 rows in all, seven remote chunks in one tile
    ("ag", 4, 64, 1, 260, 128, "bf16", {"copy_backend": "kernel", "copy_workgroups": 5}, 8),
    ("ag", 2, 4096, 8, 2048, 64, "bf16", {}, 0),      # 256 tiles: no slot left for a relay
    ("rs", 2, 200, 100, 260, 64, "bf16", {}, 0),      # 128 chunks per tile
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s-W%d-S%d-Q%d-N%d-K%d-%s-%d" % (c[:7] + (len(c[7]),)))
def test_one_shot_bit_exact(case):
    op, W, S, Q, N, K, dtype, cfg, others = case
    print("one shot", case, flush=True)
    out = "bf16" if dtype == "bf16" else "f32"
    w = si.Workload(132, "shot", op, M=W * S, N=N, K=K, dtype=dtype, out_dtype=out, dist="int", world=W, rank=W - 1,
                    shard_rows=S, chunks_per_shard=Q, order="ring" if op == "ag" else "rs_ring")
    d = si.draw(w)
    chunks, order = oracle.uniform_schedule(W, W - 1, S, Q, w.order)
    plan = csg.Plan(op, W * S, N, K, dtype, out, csg.Schedule.uniform(W, W - 1, S, Q, w.order),
                    cfg=dict(cfg, timeout_ms=1000))
    # a workgroup per unit, and eight (one per die) that relay or copy where there are any
    assert plan.info.num_workgroups == (plan.info.n_units + 7) // 8 * 8 + others
    if op == "ag":
        R = oracle.ag_gemm(d.A.device_array, d.B.device_array, chunks, order)
        for mode in ("overlap", "compute_only", "overlap"):
            c, _ = run_ag(plan, chunks, d.A, d.B, out, mode=mode, poison_remote=True, repeats=3)
            assert np.array_equal(out_to_f64(c, out), bf16_rne_of_f64(R) if out == "bf16" else R), mode
    else:
        c, o = run_rs(plan, d.A, d.B, out, repeats=3)
        R, _, _ = oracle.gemm_rs(d.A.device_array, d.B.device_array, chunks, order)
        G = out_to_f64(c, out)
        assert np.array_equal(G, bf16_rne_of_f64(R))
        O = out_to_f64(o, out)
        assert all(np.array_equal(O[x.row_begin:x.row_end], G[x.row_begin:x.row_end]) for x in chunks if not x.is_local)
    plan.close()
