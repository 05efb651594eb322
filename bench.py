"""Benchmark: float32 matmul throughput of the case-table pick over the
216-shape sweep M, N, K in {512, 1000, 2048, 3000, 4096, 8192}, against the
exhaustively-best branch, on one MI355X.

One step = one pass of the whole path over all 216 shapes: the case-table
choice for each shape (pk_select, cached per shape after its first call) and
the kernel launch (pk_matmul) on the current stream.  Inputs are resident in
HBM before timing: the operands of shape (M, N, K) are the leading M*K and K*N
elements of two 8192 x 8192 float32 buffers filled i.i.d. uniform on [-1, 1)
from seeds 0 and 1.

Prints one JSON line (rank 0, the only rank):
  value      aggregate GFLOP/s of the timed steps (2 M N K per shape)
  roofline   the kernel with the largest share of time: algorithmic flops per
             launch over its mean launch time, measured with events recorded
             around its launches inside the timed region, against the 157.3
             TFLOP/s float32 matrix-core peak
  cpu_baseline  the CPU oracle on a bounded sample of the same sweep
  exhaustive    when a tuning store for this device exists, the per-shape best
             branch timed in the same run (untimed for `value`)
  heldout    the cost model on 40 held-out shapes, every candidate timed live
  grouped    4096 uneven products in one persistent launch (a tile program
             per product), CASE and EXHAUSTIVE plans (graph replay), against
             a loop of single launches
  bf16_dense bfloat16 products at 4096^3 and 8192^3 (CASE, LEARNED and best
             program) against the 2.5 PFLOP/s bf16 matrix peak
  side       the paper's other examples (paper_1801_04348_amd/sidebench.py):
             transposition, matrix addition, 1D Jacobi, polynomial division
"""
from __future__ import annotations

import argparse
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "matmul GFLOP/s and % FP32 peak: learned/case-table pick vs exhaustive best"
FP32_PEAK_TFLOPS = 157.3
TUNED = os.path.join(ROOT, "paper_1801_04348_amd", "data", "tuned_f32_gfx950.json")
MODEL = os.path.join(ROOT, "paper_1801_04348_amd", "data", "costmodel_f32_gfx950.txt")
PROFILES = os.path.join(ROOT, "profiles")
COPY_BYTES = 256 << 20


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def cpu_baseline(budget_s: float = 15.0):
    """The oracle (float64 triple loop, OpenMP over rows) on the host cores:
    on all of them over the sweep's smallest shapes, in a fixed order, until
    about `budget_s` seconds (the reported value); single-threaded on the
    sweep's smallest shape; and the two parity configurations (float32 256^3,
    int32 1024^3) on all cores."""
    import oracle.matmul as om
    from tests import inputs
    cores = om.threads()            # before any call that sets another count

    def timed(M, N, K, dtype, nthreads, seed=0):
        if dtype == "i32":
            A = inputs.small_int_i32((M, K), seed=seed).numpy()
            B = inputs.small_int_i32((K, N), seed=seed + 1).numpy()
        else:
            A = inputs.uniform_f32((M, K), seed=seed).numpy()
            B = inputs.uniform_f32((K, N), seed=seed + 1).numpy()
        t0 = time.perf_counter()
        om.matmul(A, B, dtype, nthreads=nthreads)
        return time.perf_counter() - t0

    sample = [s for s in inputs.sweep_shapes() if max(s) <= 3000]
    flops, secs, done = 0.0, 0.0, []
    for (M, N, K) in sample:
        secs += timed(M, N, K, "f32", cores)
        flops += 2.0 * M * N * K
        done.append((M, N, K))
        if secs >= budget_s:
            break
    st = timed(512, 512, 512, "f32", 1)
    c1 = timed(256, 256, 256, "f32", cores)
    c2 = timed(1024, 1024, 1024, "i32", cores)
    return {"value": flops / secs / 1e9, "unit": "GFLOP/s", "cores": cores, "kind": "oracle",
            "sample": "%d of the sweep's shapes with M,N,K <= 3000, in sweep order, on all %d host threads "
                      "(%.1f GFLOP in %.1f s)" % (len(done), cores, flops / 1e9, secs),
            "single_thread": {"value": round(2.0 * 512 ** 3 / st / 1e9, 3), "unit": "GFLOP/s",
                              "sample": "float32 512^3, one thread (%.2f s)" % st},
            "f32_256": {"value": round(2.0 * 256 ** 3 / c1 / 1e9, 3), "unit": "GFLOP/s", "seconds": round(c1, 4)},
            "i32_1024": {"value": round(2.0 * 1024 ** 3 / c2 / 1e9, 3), "unit": "GOP/s", "seconds": round(c2, 4)}}


def heldout_section(tbl, pk, torch, inputs, Abuf, Bbuf, count=40, seed=2):
    """The learned cost model on shapes it was not trained on: the first
    `count` of the 500 held-out shapes (log-uniform on [64, 8192]^3, seed
    `seed`), operands the packed leading elements of the sweep buffers (as the
    tuner times them; rows mostly unaligned).  Per shape every feasible
    candidate is timed live (pk_measure, the EXHAUSTIVE measurement); the
    CASE pick, the model's own pick (margin 0) and the LEARNED pick (default
    5 % margin, timing near-ties itself) are scored by those timings:
    ratio = t_best / t_pick = GF_pick / GF_best."""
    import numpy as np

    def program_key(tbl, p, dtype):
        # a compiled program and its split factor: the split forms of one tile
        # program share its kernel name, and two (leaf, E) points may run one
        # instance (the fastest of their timings is the program's)
        return pk.pk_kernel_name(tbl, p, dtype), max(p.ks, 1)

    shapes = [tuple(int(x) for x in r) for r in inputs.log_uniform_shapes(500, seed)[:count]]
    Cbuf = torch.empty((max(M * N for M, N, _ in shapes),), dtype=torch.float32, device="cuda")
    t0 = time.perf_counter()
    recs = []
    for (M, N, K) in shapes:
        A = Abuf[:M * K].view(M, K)
        B = Bbuf[:K * N].view(K, N)
        C = Cbuf[:M * N].view(M, N)
        res = pk.pk_measure(tbl, "f32", M, N, K, A, B, C)
        times = {}
        for p, s in res:
            k = program_key(tbl, p, "f32")
            times[k] = min(times.get(k, s), s)
        recs.append(((M, N, K), A, B, times))
    t_measure = time.perf_counter() - t0

    def picks(policy):
        out = []
        for (shape, A, B, times) in recs:
            p = pk.pk_select_operands(tbl, "f32", A, B, policy)
            out.append(min(times.values()) / times[program_key(tbl, p, "f32")])
        return out

    def stats(r):
        r = np.sort(np.asarray(r))
        return {"geomean": round(float(np.exp(np.mean(np.log(r)))), 4), "median": round(float(np.median(r)), 4),
                "p10": round(float(np.percentile(r, 10)), 4), "worst": round(float(r[0]), 4)}

    case = picks(pk.PK_POLICY_CASE)
    pk.pk_case_table_set_learned_margin(tbl, 0.0)
    model = picks(pk.PK_POLICY_LEARNED)
    pk.pk_case_table_set_learned_margin(tbl, 0.05)
    sel0, fb0 = pk.pk_case_table_learned_stats(tbl)
    meas0 = pk.pk_case_table_learned_measured(tbl)
    learned = picks(pk.PK_POLICY_LEARNED)
    sel1, fb1 = pk.pk_case_table_learned_stats(tbl)
    meas1 = pk.pk_case_table_learned_measured(tbl)
    out = {"shapes": len(recs), "sample": "first %d of 500 shapes log-uniform on [64, 8192]^3, seed %d (disjoint "
                                          "from the training shapes), packed operands" % (count, seed),
           "candidates_per_shape": round(sum(len(r[3]) for r in recs) / len(recs), 1),
           "measure_seconds": round(t_measure, 1),
           "case": stats(case), "model_alone": stats(model), "learned": stats(learned), "learned_margin": 0.05,
           "learned_fallback_rate": round((fb1 - fb0) / max(sel1 - sel0, 1), 3),
           "learned_candidates_timed_per_fallback": round((meas1 - meas0) / max(fb1 - fb0, 1), 2)}
    out["model_alone_over_case"] = round(out["model_alone"]["geomean"] / out["case"]["geomean"], 4)
    out["learned_over_case"] = round(out["learned"]["geomean"] / out["case"]["geomean"], 4)
    return out


def bf16_section(tbl, pk, torch, inputs):
    """Dense bfloat16 products (float32 accumulate) at 4096^3 and 8192^3,
    uniform[-1,1) operands rounded to bfloat16: the CASE pick, the LEARNED
    pick (where the table has a bfloat16 model) and the exhaustively-best
    program, against the 2.5 PFLOP/s dense bf16 matrix peak."""
    out = {}
    for n in (4096, 8192):
        A = inputs.bf16_bits(inputs.uniform_f32((n, n), seed=21)).cuda()
        B = inputs.bf16_bits(inputs.uniform_f32((n, n), seed=22)).cuda()
        C = torch.empty((n, n), dtype=torch.float32, device="cuda")
        row = {}
        for name, pol in (("case", pk.PK_POLICY_CASE), ("learned", pk.PK_POLICY_LEARNED),
                          ("best", pk.PK_POLICY_EXHAUSTIVE)):
            try:
                p = pk.pk_select(tbl, "bf16", n, n, n, pol)
            except pk.PkError as e:
                if e.code == pk.PK_ERR_COST_MODEL:
                    continue
                raise
            reps = 100 if n <= 4096 else 20  # tens of milliseconds per measurement
            # warm-up of about a quarter second: the shader clock settles under
            # a sustained bf16 load (short warm-ups read up to 10 % apart)
            t0 = time.perf_counter()
            while time.perf_counter() - t0 < 0.25:
                for _ in range(reps // 4):
                    pk.pk_matmul(tbl, p, "bf16", A, B, C)
                torch.cuda.synchronize()
            times = []
            for _ in range(3):  # the median of three measurements
                e0 = torch.cuda.Event(enable_timing=True)
                e1 = torch.cuda.Event(enable_timing=True)
                e0.record()
                for _ in range(reps):
                    pk.pk_matmul(tbl, p, "bf16", A, B, C)
                e1.record()
                torch.cuda.synchronize()
                times.append(e0.elapsed_time(e1) / reps * 1e-3)
            s = sorted(times)[1]
            row[name] = {"kernel": pk.pk_kernel_name(tbl, p, "bf16"), "tflops": round(2.0 * n ** 3 / s / 1e12, 1),
                         "pct_bf16_peak": round(2.0 * n ** 3 / s / 2.5e15, 4)}
        out["%dx%dx%d" % (n, n, n)] = row
    return out


def grouped_section(tbl, pk, torch, inputs, dtype, reps=5):
    """4096 independent products, M, N, K each round(exp(U(ln 16, ln 512)))
    from seed 0, operands packed in three buffers with rows padded to 8
    elements (workloads.grouped_operands): one grouped plan (CASE, and the
    EXHAUSTIVE auto-tuner's) replayed from its captured graph, against a loop
    of 4096 single-product launches (eager, and captured in a graph)."""
    import numpy as np
    from paper_1801_04348_amd import workloads
    G = 4096
    dims, As, Bs, Cs = workloads.grouped_operands(torch, inputs, dtype, G=G)
    flops = float(2 * np.prod(dims.astype(np.float64), axis=1).sum())
    es = 2 if dtype == "bf16" else 4
    peak = 2.5e15 if dtype == "bf16" else 157.3e12
    per_bytes = es * (dims[:, 0] * dims[:, 2] + dims[:, 2] * dims[:, 1]) + 4.0 * dims[:, 0] * dims[:, 1]
    roof = float(np.sum(np.maximum(2.0 * np.prod(dims.astype(np.float64), axis=1) / peak, per_bytes / 8e12)))

    def timed(fn):
        # a quarter second of untimed runs first: the clock settles under the
        # load (a plan timed right after the device sat idle runs 10-20 %
        # slower than in steady state)
        t0 = time.perf_counter()
        while True:
            fn()
            torch.cuda.synchronize()
            if time.perf_counter() - t0 >= 0.25:
                break
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / reps * 1e-3

    plan = pk.pk_grouped_plan_create(tbl, dtype, As, Bs, Cs, policy=pk.PK_POLICY_CASE)
    n_launch, tiles, chosen = plan.info()
    plan.capture()
    t_graph = timed(lambda: plan.replay())
    t_plan = timed(lambda: plan.run())
    # the program chosen by timing each candidate plan on these operands
    plan_x = pk.pk_grouped_plan_create(tbl, dtype, As, Bs, Cs, policy=pk.PK_POLICY_EXHAUSTIVE)
    chosen_x = plan_x.info()[2]
    tiles_of = lambda ch: sorted({"%dx%d" % (c.bm, c.bn) for c in ch})  # noqa: E731
    plan_x.capture()
    t_graph_x = timed(lambda: plan_x.replay())
    picks = [pk.pk_select(tbl, dtype, int(M), int(N), int(K), pk.PK_POLICY_CASE) for (M, N, K) in dims]

    def loop():
        for g in range(G):
            pk.pk_matmul(tbl, picks[g], dtype, As[g], Bs[g], Cs[g])
    t_loop = timed(loop)
    graph = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        loop()
    torch.cuda.current_stream().wait_stream(s)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        loop()
    t_loop_graph = timed(lambda: graph.replay())
    return {"products": G, "gflop": round(flops / 1e9, 2), "launches": n_launch, "tiles": tiles,
            "kernels": plan.kernels(), "tile_programs": tiles_of(chosen),
            "grouped_graph_gflops": round(flops / t_graph / 1e9, 1),
            "exhaustive_kernels": plan_x.kernels(), "exhaustive_tile_programs": tiles_of(chosen_x),
            "exhaustive_launches": plan_x.info()[0],
            "exhaustive_graph_gflops": round(flops / t_graph_x / 1e9, 1),
            "exhaustive_pct_summed_roofline": round(roof / t_graph_x, 4),
            "grouped_gflops": round(flops / t_plan / 1e9, 1),
            "loop_gflops": round(flops / t_loop / 1e9, 1),
            "loop_graph_gflops": round(flops / t_loop_graph / 1e9, 1),
            "speedup_vs_loop": round(t_loop / t_graph, 2),
            "speedup_vs_loop_graph": round(t_loop_graph / t_graph, 2),
            "pct_summed_roofline": round(roof / t_graph, 4)}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--policy", choices=["auto", "case", "learned"], default="auto",
                    help="auto: the learned cost model when one for this machine is shipped, else the case table")
    ap.add_argument("--sweep-only", action="store_true",
                    help="run the timed sweep only: skip the untimed sections (exhaustive comparison, grouped "
                         "products, side benchmarks), e.g. for a profile of the sweep's kernels alone")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-heldout", action="store_true", help="skip the held-out cost-model section")
    ap.add_argument("--per-shape", default=None,
                    help="write each sweep shape's program and one-launch time of the untimed pass (JSON)")
    ap.add_argument("--machine", default=None,
                    help="bind the case table to this recorded machine descriptor (JSON) instead of the runtime's")
    ap.add_argument("--save-machine", default=None, help="write the machine descriptor the table was bound to")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="run a 256 MiB device copy three times first (known bytes, for counter calibration), then "
                         "once right before and once right after the timed steps (they delimit the timed "
                         "region's dispatches in a profile; see paper_1801_04348_amd/profwindow.py)")
    ap.add_argument("--save-picks", default=None, help="write the program chosen for each sweep shape (JSON)")
    ap.add_argument("--load-picks", default=None,
                    help="run the programs a previous run chose (its --save-picks file) instead of selecting: "
                         "profiling runs then time the same launches as that run")
    args = ap.parse_args()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py measures one GPU only: the product path has no multi-GPU part; run with --gpus 1",
              file=sys.stderr)
        sys.exit(2)

    import torch

    from paper_1801_04348_amd import pk
    from tests import inputs

    torch.cuda.init()
    if args.machine:
        with open(args.machine) as f:
            tbl = pk.pk_case_table_build(0, pk.machine(**json.load(f)))
    else:
        tbl = pk.pk_case_table_build(0)
    machine = pk.pk_case_table_describe(tbl)["machine"]
    if args.save_machine:
        with open(args.save_machine, "w") as f:
            json.dump(machine, f)
    model_note = None
    have_model = False
    if args.policy in ("auto", "learned") and os.path.exists(MODEL):
        try:
            pk.pk_case_table_set_costmodel(tbl, pk.pk_costmodel_load(MODEL))
            have_model = True
        except pk.PkError as e:
            model_note = str(e)
        if have_model:
            pk.load_shipped_models(tbl)  # the other element types' models, for the side sections
    if args.policy == "learned" and not have_model:
        sys.exit("no usable cost model: %s" % (model_note or MODEL))
    policy_name = "learned" if have_model and args.policy != "case" else "case"
    policy = pk.PK_POLICY_LEARNED if policy_name == "learned" else pk.PK_POLICY_CASE
    if args.load_picks:
        policy_name = "picks of a previous run (%s)" % os.path.basename(args.load_picks)
    shapes = inputs.sweep_shapes()
    big = max(max(s) for s in shapes)
    Abuf = inputs.uniform_f32((big * big,), seed=0).cuda()
    Bbuf = inputs.uniform_f32((big * big,), seed=1).cuda()
    Cbuf = torch.empty((big * big,), dtype=torch.float32, device="cuda")
    marker = None
    if args.calibrate_copy:
        # no fill kernel: the five adds are the only non-library kernels of
        # that size (their values do not matter)
        src_t = torch.empty(COPY_BYTES // 4, dtype=torch.float32, device="cuda")
        dst_t = torch.empty_like(src_t)

        def marker():
            torch.add(src_t, 0.0, out=dst_t)

        for _ in range(3):
            marker()
        torch.cuda.synchronize()
    ops = []
    picks = None
    if args.load_picks:
        with open(args.load_picks) as f:
            picks = {tuple(r["shape"]): pk.params(**r["params"]) for r in json.load(f)}
    for (M, N, K) in shapes:
        p = picks[(M, N, K)] if picks else pk.pk_select(tbl, "f32", M, N, K, policy, allow_fallback=True)
        ops.append(dict(M=M, N=N, K=K, A=Abuf[:M * K].view(M, K), B=Bbuf[:K * N].view(K, N),
                        C=Cbuf[:M * N].view(M, N), p=p, name=pk.pk_kernel_name(tbl, p, "f32"),
                        flops=2.0 * M * N * K))
    flops_step = sum(o["flops"] for o in ops)
    if args.save_picks:
        with open(args.save_picks, "w") as f:
            json.dump([{"shape": [o["M"], o["N"], o["K"]], "params": o["p"].as_dict()} for o in ops], f)

    def one_pass(events=None):
        for o in ops:
            p = o["p"] if picks else pk.pk_select(tbl, "f32", o["M"], o["N"], o["K"], policy, allow_fallback=True)
            if events is not None and o["name"] == dominant:
                e0, e1 = events.pop()
                e0.record()
                pk.pk_matmul(tbl, p, "f32", o["A"], o["B"], o["C"])
                e1.record()
                recorded.append((o, e0, e1))
            else:
                pk.pk_matmul(tbl, p, "f32", o["A"], o["B"], o["C"])

    # warm-up, then one untimed pass with events around every launch to find
    # the kernel holding the largest share of the time
    for _ in range(max(args.warmup, 1)):
        one_pass()
    torch.cuda.synchronize()
    share = {}
    evs = []
    for o in ops:
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        e0.record()
        pk.pk_matmul(tbl, o["p"], "f32", o["A"], o["B"], o["C"])
        e1.record()
        evs.append((o, e0, e1))
    torch.cuda.synchronize()
    per_shape_ms = {}
    for o, e0, e1 in evs:
        ms = e0.elapsed_time(e1)
        per_shape_ms[(o["M"], o["N"], o["K"])] = ms
        share[o["name"]] = share.get(o["name"], 0.0) + ms
    if args.per_shape:
        with open(args.per_shape, "w") as f:
            json.dump([{"shape": [o["M"], o["N"], o["K"]], "kernel": o["name"],
                        "ms": per_shape_ms[(o["M"], o["N"], o["K"])],
                        "tflops": o["flops"] / per_shape_ms[(o["M"], o["N"], o["K"])] / 1e9} for o in ops], f)
    dominant = max(share, key=share.get)
    n_dom = sum(1 for o in ops if o["name"] == dominant)
    log("dominant kernel %s: %.1f%% of launch time, %d launches per step"
        % (dominant, 100 * share[dominant] / sum(share.values()), n_dom))

    # timed region
    pool = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
            for _ in range(n_dom * args.steps)]
    recorded = []
    if marker:
        marker()  # the fourth copy: the timed region's launches follow it
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        one_pass(pool)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    if marker:
        marker()  # the fifth copy closes the window
        torch.cuda.synchronize()
    value = flops_step * args.steps / elapsed / 1e9
    dom_flops = sum(o["flops"] for o, _, _ in recorded)
    dom_bytes = sum(4.0 * (o["M"] * o["K"] + o["K"] * o["N"] + o["M"] * o["N"]) for o, _, _ in recorded)
    dom_s = sum(e0.elapsed_time(e1) for _, e0, e1 in recorded) * 1e-3
    achieved = dom_flops / dom_s / 1e12
    roofline = {"bound": "mfma", "kernel": dominant, "achieved": round(achieved, 2), "peak": FP32_PEAK_TFLOPS,
                "unit": "TFLOP/s", "frac": round(achieved / FP32_PEAK_TFLOPS, 4), "traffic": None,
                "launches": len(recorded), "mean_launch_us": round(dom_s / len(recorded) * 1e6, 2),
                "flops_per_launch": dom_flops / len(recorded),
                "algorithmic_bytes_per_launch": dom_bytes / len(recorded)}
    # HBM bytes per launch of this kernel from the counter passes, if they
    # were taken on the current kernel source (see paper_1801_04348_amd/traffic.py)
    from paper_1801_04348_amd import traffic as trf
    tr_path = os.path.join(PROFILES, "traffic_%s.json" % dominant)
    if os.path.exists(tr_path):
        with open(tr_path) as f:
            tr = json.load(f)
        if tr.get("kernel") == dominant and tr.get("source_sha256") == trf.kernel_source_hash():
            roofline["traffic"] = tr["bytes_per_launch"]
            roofline["traffic_over_algorithmic"] = round(tr["bytes_per_launch"] / roofline["algorithmic_bytes_per_launch"], 3)

    # large shapes and the exhaustive comparison (untimed for `value`)
    large = {}
    for s in [(4096, 4096, 4096), (8192, 8192, 8192)]:
        ms = per_shape_ms[s]
        large["x".join(map(str, s))] = {"gflops": round(2.0 * s[0] * s[1] * s[2] / ms / 1e6, 1),
                                         "pct_fp32_peak": round(2.0 * s[0] * s[1] * s[2] / ms / 1e9 / FP32_PEAK_TFLOPS, 4)}
    # per shape, interleaved: the exhaustively-best branch (tuning store of this
    # machine), the CASE pick and the LEARNED pick (untimed for `value`)
    exhaustive = None
    best = {}
    if os.path.exists(TUNED) and not args.sweep_only:
        with open(TUNED) as f:
            tuned = json.load(f)
        if tuned["machine"]["regs_block"] == machine["regs_block"]:
            best = {tuple(r["shape"]): pk.params(**r["params"]) for r in tuned["shapes"]}
    if best:
        def t_of(p, o, reps=3):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            pk.pk_matmul(tbl, p, "f32", o["A"], o["B"], o["C"])
            e[0].record()
            for _ in range(reps):
                pk.pk_matmul(tbl, p, "f32", o["A"], o["B"], o["C"])
            e[1].record()
            torch.cuda.synchronize()
            return e[0].elapsed_time(e[1]) / reps
        tot = {"best": 0.0, "case": 0.0, "learned": 0.0}
        ratios = {"case": [], "learned": []}
        fl = 0.0
        for o in ops:
            key = (o["M"], o["N"], o["K"])
            if key not in best:
                continue
            fl += o["flops"]
            tb = t_of(best[key], o)
            tc = t_of(pk.pk_select(tbl, "f32", *key, pk.PK_POLICY_CASE), o)
            tl = t_of(pk.pk_select(tbl, "f32", *key, pk.PK_POLICY_LEARNED), o) if have_model else tc
            # the best of this run's three timings: the tuner's stored best
            # need not be the fastest on this box today
            tb = min(tb, tc, tl)
            tot["best"] += tb
            tot["case"] += tc
            ratios["case"].append(tb / tc)
            if have_model:
                tot["learned"] += tl
                ratios["learned"].append(tb / tl)
        geo = lambda r: round(math.exp(sum(map(math.log, r)) / len(r)), 4)
        exhaustive = {"shapes": len(ratios["case"]),
                      "sample": "the float32 model was trained on random shapes of the same range, not on these "
                                "shapes; best = the fastest of the tuner's stored pick, CASE and LEARNED, timed "
                                "interleaved in this run",
                      "best_gflops": round(fl / tot["best"] / 1e6, 1),
                      "case_gflops": round(fl / tot["case"] / 1e6, 1),
                      "case_over_best_geomean": geo(ratios["case"]), "case_over_best_min": round(min(ratios["case"]), 4)}
        if have_model:
            sel, fb = pk.pk_case_table_learned_stats(tbl)
            exhaustive.update({"learned_gflops": round(fl / tot["learned"] / 1e6, 1),
                               "learned_over_best_geomean": geo(ratios["learned"]),
                               "learned_over_best_min": round(min(ratios["learned"]), 4),
                               "learned_fallback_rate": round(fb / max(sel, 1), 3)})

    heldout = None
    if have_model and not args.sweep_only and not args.no_heldout:
        heldout = heldout_section(tbl, pk, torch, inputs, Abuf, Bbuf)
        log("held-out: %s" % json.dumps(heldout))
    side = None
    if not args.sweep_only:
        from paper_1801_04348_amd import sidebench
        side = sidebench.run_all(tbl, pk, torch, inputs)
    grouped = None
    bf16 = None
    if not args.sweep_only:
        grouped = {dt: grouped_section(tbl, pk, torch, inputs, dt) for dt in ("f32", "bf16")}
        bf16 = bf16_section(tbl, pk, torch, inputs)

    out = {"metric": METRIC, "value": round(value, 1), "unit": "GFLOP/s", "n_gpus": 1, "steps": args.steps,
           "warmup": args.warmup, "ms_per_step": round(elapsed / args.steps * 1e3, 3), "higher_is_better": True,
           "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
           "config": {"workload": "fp32 matmul sweep, M,N,K in {512,1000,2048,3000,4096,8192} (216 shapes), "
                                  "uniform[-1,1) operands, %s pick per shape" % policy_name,
                      "shapes": len(shapes), "gflop_per_step": round(flops_step / 1e9, 1), "policy": policy_name,
                      "parallelism": "none (1 GPU)"},
           "pct_fp32_peak": round(value / 1e3 / FP32_PEAK_TFLOPS, 4),
           "large_shapes": large, "exhaustive": exhaustive, "heldout": heldout, "grouped": grouped, "bf16_dense": bf16, "side": side,
           "roofline": roofline,
           "machine": {k: machine[k] for k in ("arch", "cu_count", "lds_block", "regs_block", "max_blocks_cu")}}
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline()
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
