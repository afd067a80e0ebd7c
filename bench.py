#!/usr/bin/env python3
"""Planner benchmark on one MI355X.

One step = one plan of the sampling MPC planner: the HIP rollout of K
candidate control sequences through the single-rigid-body model over the
heightmap (stage cost and ESM constraint at every Euler step), followed by
the argmin selection and the 8-byte readback of (k*, J*) -- what one MPC
iteration needs before it can act. The default workload is the stress
rollout: a single plan of K=65536 candidates x N=200 steps (dt 0.01 s) over a
2048x2048 terrain at 0.05 m with alternating 15-degree side slopes, 0.5 m
berms and 0.3 m ruts, initial speed 20 m/s (synthetic, seeded). The
single-plan workload (K=4096, N=100, 512x512) is reported as a row.

Prints one JSON line: rollout-steps/s (K*N*substeps per plan / wall time per
plan), p50/p99 plan latency (over at least 100 plans), the rollout kernel's
ALU roofline fraction (HIP events on the planner's stream) and the FP64
oracle timed on the host cores on a bounded sample of the same workload.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

METRIC = "candidate rollout-steps/sec and p50/p99 plan latency (serving vs plain)"

# FP32 operations per rollout-step of the step definition, one lane per
# candidate, transcendentals counted as one: goal test 5, attitude 21, CoM in
# grid units 2, kinematics 24, the four wheels' contact points and lookup
# coordinates 21 and contact velocities 13 (the lever arms share their
# front/rear and left/right terms), per wheel 59 (cell index and weights 9,
# interpolation of four channels from the cell's bilinear coefficients 12,
# normal 6, extension 3, rate 6, spring and damper 7, slip 6, tire 5, forces
# and the moment terms rx Fz and rx fy 5), wheel sums 18, the three moments
# from those sums 4, right-hand side rows 17, ESM and soft cost 12, running
# cost 5, Euler update and clamps 19, control clamp 5 per interval: 402 with
# a costmap. A plan without a costmap has no cost-channel term (its
# interpolation at the four wheels 12, its wheel sum 3 and its addition to
# the running cost 1), and its kernels skip it: 386. Every workload here runs
# without a costmap, so the algorithmic side of the ALU roofline counts 386.
OPS_PER_STEP_COSTMAP = 402
OPS_PER_STEP = OPS_PER_STEP_COSTMAP - 16
# MI355X vector ALU issue: 256 CUs x 4 SIMD x 16 lanes x 2.4 GHz, one
# non-packed FP32 operation per lane per clock.
ALU_PEAK_GOPS = 256 * 4 * 16 * 2.4
# HBM bytes per launch of the fused rollout kernel, from rocprofv3
# FETCH_SIZE / WRITE_SIZE (KiB per dispatch, one `--pmc` run each over this
# script with `--steps 10 --warmup 2 --cpu-seconds 0 --serving 0 --rows 0`)
# scaled by what the same counters read for a 256 MiB device copy
# (`--calibrate-copy 256`). Each entry records the signature of the rollout
# sources and build flags it was taken on (kernel_signature()); once they
# change, the figure no longer describes the kernel and is reported as null.
# workload: (FETCH_SIZE KiB, WRITE_SIZE KiB, fetch scale, write scale, signature)
TRAFFIC_COUNTERS = {
    # fused kernel, one lane per candidate (c5, 256-thread workgroups) and four
    # lanes (c2, 64), no costmap, cell-coefficient terrain; copy calibration
    # 262144 KiB read as 131084.44 KiB (x1.99981) and written as 262144.0 KiB (x1.0)
    "c5": (60620.14, 273.69, 262144.0 / 131084.44, 1.0, "4f6a3fe22f778b4b"),
    "c2": (4979.88, 32.91, 262144.0 / 131084.44, 1.0, "4f6a3fe22f778b4b"),
}
ROLLOUT_SOURCES = ("rollout_step.h", "rollout_kernels.h", "rollout.hip",
                   "rollout_onelane_1wave.hip", "rollout_multilane.hip",
                   "rollout_multilane_1wave.hip", "plan_internal.h",
                   "select_common.h", "sample.h")


def kernel_signature():
    """First 16 hex digits of a SHA-256 over the rollout kernel's sources and
    the library's build script (its compiler flags)."""
    import hashlib
    h = hashlib.sha256()
    pkg = os.path.join(ROOT, "paper_2603_20525_amd")
    for name in ROLLOUT_SOURCES:
        with open(os.path.join(pkg, "csrc", name), "rb") as f:
            h.update(name.encode() + b"\0" + f.read())
    with open(os.path.join(pkg, "build.py"), "rb") as f:
        h.update(f.read())
    return h.hexdigest()[:16]


def traffic_bytes(workload_name):
    """Counter-derived HBM bytes per launch, or None when no counters were
    taken on the current kernel for this workload."""
    t = TRAFFIC_COUNTERS.get(workload_name)
    if t is None or t[4] != kernel_signature():
        return None
    fetch_kib, write_kib, fs, ws, _ = t
    return (fetch_kib * fs + write_kib * ws) * 1024.0


def workload(name):
    from paper_2603_20525_amd import inputs
    if name == "c2":
        return inputs.c2(), "single plan: K=4096 candidates, N=100 steps at dt=0.02 s, " \
                            "512x512 fBm+berms terrain at 0.1 m, v0=15 m/s"
    if name == "c5":
        return inputs.c5(), "stress: K=65536, N=200 at dt=0.01 s, 2048x2048 side-slope/berm/rut " \
                            "terrain at 0.05 m, v0=20 m/s"
    if name == "paper":
        return inputs.paper_shape(), "paper solver shape: K=204288 uniform samples, 16 ZOH x 0.25 s, " \
                                     "50 Euler substeps (5 ms), paper vehicle, 512x512 terrain"
    raise SystemExit(f"unknown workload {name}")


def percentile(xs, q):
    s = sorted(xs)
    if not s:
        return None
    i = min(len(s) - 1, max(0, int(round(q / 100.0 * (len(s) - 1)))))
    return s[i]


def cpu_baseline(w, seconds):
    """FP64 oracle on the host cores: full rollouts of the same workload
    (or a candidate subset for very large K), repeated for about `seconds`."""
    import numpy as np
    import oracle
    threads = int(os.environ.get("OMP_NUM_THREADS") or len(os.sched_getaffinity(0)))
    o = oracle.Oracle(w.vehicle, w.cost, w.integ)
    T = w.terrain
    o.set_terrain(T.height, T.x0, T.y0, T.res)
    K = w.K
    u = w.controls
    sample = f"full workload (K={K}, N={w.N})"
    if K > 8192:
        idx = np.arange(0, K, K // 4096)[:4096]
        u = np.ascontiguousarray(u[:, :, idx])
        sample = f"{len(idx)}-candidate subset of K={K}, N={w.N}"
    steps_per_run = u.shape[2] * u.shape[0] * w.integ["substeps"]
    runs, t0 = 0, time.perf_counter()
    while True:
        o.rollout(w.state0, u)
        runs += 1
        el = time.perf_counter() - t0
        if el >= seconds or runs >= 1000:
            break
    out = {"value": steps_per_run * runs / el, "unit": "rollout-steps/s", "cores": threads,
           "kind": "oracle",
           "sample": f"{sample} repeated {runs}x in {el:.1f} s (FP64 C, OpenMP over candidates)"}
    # the same oracle on one core (OpenMP team of one; a quarter of the time budget)
    import ctypes
    gomp = ctypes.CDLL("libgomp.so.1")
    gomp.omp_set_num_threads(1)
    try:
        runs1, t1 = 0, time.perf_counter()
        while True:
            o.rollout(w.state0, u)
            runs1 += 1
            el1 = time.perf_counter() - t1
            if el1 >= seconds / 4 or runs1 >= 1000:
                break
    finally:
        gomp.omp_set_num_threads(threads)
    out["single_thread"] = {"value": steps_per_run * runs1 / el1, "cores": 1,
                            "sample": f"{sample} repeated {runs1}x in {el1:.1f} s"}
    return out


def _summ(lat, t_first, t_last, steps, n):
    span = max(t_last - t_first, 1e-9)
    return {"p50_ms": percentile(lat, 50) * 1e3, "p99_ms": percentile(lat, 99) * 1e3,
            "max_ms": max(lat) * 1e3, "req_per_s": n / span, "rollout_steps_per_s": steps / span}


# Algorithmic FP32 operations per step of the other rollout variants (same
# counting rules as OPS_PER_STEP). EST: the cell under the CoM, its lookup
# coordinates and the interpolation of two channels (f_x, f_y) 19, angles
# from the normal 10, sincos psi, rotation and
# world velocity 16, load transfer 6, two slip angles 10, tires 12, rows,
# constraint and cost 20, Euler and limits 12, goal test 5. RK4: four
# right-hand sides, the stage and combination updates, one set of limits.
EST_OPS_PER_STEP = 109
RK4_OPS_PER_STEP = 4 * (OPS_PER_STEP - 24) + 24 + 3 * 13 * 2 + 2 * 13
# Adjoint, per candidate-step (same rules, no costmap): the checkpointing
# forward pass runs the Euler step (OPS_PER_STEP); the backward kernel
# recomputes the step from its segment's checkpoint (OPS_PER_STEP) and
# evaluates the step's vector-Jacobian product: its forward quantities
# (attitude and chassis 45, CoM in grid units 2, the four wheels' contact
# points, lookup coordinates and velocities 34, four wheels of 96: gathers,
# slip, normal, suspension, tire) and the reverse sweep (chassis rows,
# rotation, trigonometry 160; four wheels of 107, the cost channel's
# cell-weight derivatives left out; wheel sums 63), 1 116 in all.
ADJ_VJP_OPS_PER_STEP = 45 + 2 + 34 + 4 * 96 + 160 + 4 * 107 + 63
ADJ_BWD_OPS_PER_STEP = OPS_PER_STEP + ADJ_VJP_OPS_PER_STEP
HBM_PEAK_GBS = 8000.0


def _time_ms(fn, reps=5, warm=2):
    """Median duration (ms) of fn() between HIP events on the current stream."""
    import torch
    for _ in range(warm):
        fn()
    ts = []
    for _ in range(reps):
        a = torch.cuda.Event(enable_timing=True)
        b = torch.cuda.Event(enable_timing=True)
        a.record()
        fn()
        b.record()
        torch.cuda.synchronize()
        ts.append(a.elapsed_time(b))
    ts.sort()
    return ts[len(ts) // 2]


def rows_leg():
    """One measurement per widened row of the path, each against its bound:
    the paper's own solver shape end to end (in-kernel sampling, rollout and
    argmin in one launch), the extended single-track baseline, the RK4
    option, the adjoint, and the terrain preparation kernels."""
    import numpy as np
    import torch
    from paper_2603_20525_amd import inputs
    from paper_2603_20525_amd import plan as P
    out = {}
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()  # noqa: E731
    alu = lambda ops, sec: ops / sec / 1e9 / ALU_PEAK_GOPS  # noqa: E731

    # paper shape: K = 204 288 uniform steering-rate samples, 16 x 0.25 s, 5 ms Euler
    T = inputs.fbm_berm_terrain(2000)
    w = inputs.paper_shape(K=8, terrain=T)
    K, N, S = 204288, 16, w.integ["substeps"]
    pl = P.Planner(w.vehicle, w.cost, w.integ, K, N, T.W, T.H)
    pl.set_terrain(dev(T.height), T.x0, T.y0, T.res)
    spec = P.sample_spec(P.PLAN_SAMPLE_UNIFORM, 6000, 0, (1.0, 0.0))
    J = torch.empty(K, device="cuda")
    plan = torch.empty(N, 2, device="cuda")
    plan_call = lambda: pl.rollout_sampled_argmin(w.state0, spec, N, J, plan,  # noqa: E731
                                                   want_result=False)
    # default: the candidates run in locality order (sorting included)
    ms = _time_ms(plan_call)
    ordered = pl.get_order()
    pl.set_order(P.PLAN_ORDER_OFF)
    ms_unordered = _time_ms(plan_call)
    pl.set_order(P.PLAN_ORDER_AUTO)
    steps = K * N * S
    out["paper_shape_sampled_one_launch"] = {
        "ms_per_plan": ms, "plans_per_s": 1e3 / ms, "samples_per_s": K * 1e3 / ms,
        "rollout_steps_per_s": steps * 1e3 / ms, "alu_frac": alu(OPS_PER_STEP * steps, ms / 1e3),
        "locality_order": ordered, "ms_per_plan_unordered": ms_unordered,
        "paper_context": "11e6 samples/s (80 Hz) on an RTX 5000 Ada Mobile; about 21e6 on an "
                         "RTX 6000 Ada (other hardware, scanned terrain)"}
    # materialised samples of the same shape (generator only: 2 N K floats written)
    u = torch.empty(N, 2, K, device="cuda")
    ms = _time_ms(lambda: pl.sample_controls(spec, u))
    nbytes = 8 * N * K
    out["sample_controls_paper_shape"] = {"ms": ms, "gb_per_s": nbytes / ms / 1e6,
                                          "hbm_frac": nbytes / ms / 1e6 / HBM_PEAK_GBS}
    # extended single-track formulation at the same shape (materialised samples)
    s13 = w.state0
    s7 = [s13[0], s13[1], s13[3], s13[7], s13[11], s13[12], s13[6]]
    # materialised controls are ordered on request (the automatic mode orders
    # in-kernel uniform draws only); both orders are reported
    pl.set_order(P.PLAN_ORDER_ON)
    ms_est = _time_ms(lambda: pl.rollout_est(s7, u, J))
    ms_srb = _time_ms(lambda: pl.rollout(w.state0, u, J))
    pl.set_order(P.PLAN_ORDER_OFF)
    ms_est_u = _time_ms(lambda: pl.rollout_est(s7, u, J))
    ms_srb_u = _time_ms(lambda: pl.rollout(w.state0, u, J))
    pl.set_order(P.PLAN_ORDER_AUTO)
    # the row reports the faster order (both are given)
    best = min(ms_est, ms_est_u)
    out["est_paper_shape"] = {
        "ms": best, "locality_order": bool(ms_est < ms_est_u),
        "rollout_steps_per_s": steps * 1e3 / best,
        "alu_frac": alu(EST_OPS_PER_STEP * steps, best / 1e3),
        "ms_ordered": ms_est, "ms_unordered": ms_est_u,
        "srb_ms_same_samples": ms_srb, "srb_ms_same_samples_unordered": ms_srb_u}
    pl.close()

    # RK4 on the single-plan workload
    w = inputs.c2()
    w.integ = dict(w.integ, method=P.PLAN_RK4)
    pl = P.Planner(w.vehicle, w.cost, w.integ, w.K, w.N, w.terrain.W, w.terrain.H)
    pl.set_terrain(dev(w.terrain.height), w.terrain.x0, w.terrain.y0, w.terrain.res)
    uc = dev(w.controls)
    Jc = torch.empty(w.K, device="cuda")
    ms = _time_ms(lambda: pl.rollout(w.state0, uc, Jc))
    steps = w.K * w.N
    out["rk4_single_plan"] = {"ms": ms, "rollout_steps_per_s": steps * 1e3 / ms,
                              "alu_frac": alu(RK4_OPS_PER_STEP * steps, ms / 1e3)}
    pl.close()

    # softmin selection on the single-plan workload: weights over all K
    # costs, weighted mean of all K control sequences (HBM: the controls and
    # costs read once, the plan written)
    w = inputs.c2()
    pl = P.Planner(w.vehicle, w.cost, w.integ, w.K, w.N, w.terrain.W, w.terrain.H)
    pl.set_terrain(dev(w.terrain.height), w.terrain.x0, w.terrain.y0, w.terrain.res)
    uc = dev(w.controls)
    Jc = torch.empty(w.K, device="cuda")
    pc = torch.empty(w.N, 2, device="cuda")
    pl.rollout(w.state0, uc, Jc)
    ms = _time_ms(lambda: pl.select(uc, Jc, pc, mode=P.PLAN_SOFTMIN, lam=10.0,
                                    want_result=False), reps=20, warm=5)
    nbytes = 4 * (2 * w.N * w.K + w.K + 2 * w.N)
    out["softmin_select_single_plan"] = {"ms": ms, "bytes": nbytes,
                                         "gb_per_s": nbytes / (ms / 1e3) / 1e9,
                                         "hbm_frac": nbytes / (ms / 1e3) / 1e9 / HBM_PEAK_GBS}
    pl.close()

    # adjoint: forward (checkpoints every 10 intervals) + backward, K = 1024
    # and the top-32 refinement set
    w = inputs.c4()
    pl = P.Planner(w.vehicle, w.cost, w.integ, w.K, w.N, w.terrain.W, w.terrain.H)
    pl.set_terrain(dev(w.terrain.height), w.terrain.x0, w.terrain.y0, w.terrain.res)
    res = {"ops_per_step": {"forward": OPS_PER_STEP, "backward": ADJ_BWD_OPS_PER_STEP}}
    for name, Kk in (("K1024", w.K), ("top32", 32)):
        uk = dev(np.ascontiguousarray(w.controls[:, :, :Kk]))
        Jk = torch.empty(Kk, device="cuda")
        gk = torch.empty_like(uk)
        msg = _time_ms(lambda: pl.rollout_grad(w.state0, uk, Jk, gk, checkpoint_every=10))
        # the backward kernel alone: HIP events on the planner's stream
        pl.enable_timing(True)
        bwd = []
        for _ in range(5):
            pl.rollout_grad(w.state0, uk, Jk, gk, checkpoint_every=10)
            bwd.append(pl.last_rollout_ms())
        pl.enable_timing(False)
        bwd.sort()
        ms_b = bwd[len(bwd) // 2]
        steps = Kk * w.N
        res[name] = {"ms": msg, "forward_steps_per_s": steps * 1e3 / msg,
                     "alu_frac": alu((OPS_PER_STEP + ADJ_BWD_OPS_PER_STEP) * steps, msg / 1e3),
                     "backward_kernel_ms": ms_b,
                     "backward_alu_frac": alu(ADJ_BWD_OPS_PER_STEP * steps, ms_b / 1e3),
                     "launch": list(pl.get_launch())}
    out["adjoint_c4"] = res
    pl.close()

    # terrain preparation on the 2048 x 2048 map: level-of-detail smoothing
    # (HBM: two passes, each reading and writing the grid once) and the costmap
    T = inputs.side_slope_terrain(5000)
    pl = P.Planner(inputs.WORKLOAD_VEHICLE, inputs.BASE_COST, inputs.BASE_INTEG, 8, 8, T.W, T.H)
    h = dev(T.height)
    o_ = torch.empty_like(h)
    sm = {}
    for sigma in (0.3, 1.5):
        ms = _time_ms(lambda: pl.smooth_terrain(h, T.res, sigma, o_))
        r = int(np.ceil(3 * sigma / T.res - 1e-6))
        nbytes = 2 * 2 * 4 * T.W * T.H
        sm[f"sigma_{sigma}"] = {
            "ms": ms, "taps": 2 * r + 1, "gb_per_s": nbytes / ms / 1e6,
            "hbm_frac": nbytes / ms / 1e6 / HBM_PEAK_GBS,
            "alu_frac": alu(2 * (2 * r + 1) * T.W * T.H, ms / 1e3)}
    out["lod_smoothing_2048"] = sm
    polys = inputs.obstacle_polygons(T, seed=5, count=20, boundary=True)
    verts = np.concatenate([np.asarray(v, np.float32).reshape(-1, 2) for _, v in polys])
    offsets = np.concatenate([[0], np.cumsum([len(v) for _, v in polys])]).astype(int)
    kinds = [k for k, _ in polys]
    vd = dev(verts)
    cm = torch.empty_like(h)
    ms = _time_ms(lambda: pl.costmap_polygons(vd, offsets, kinds, cm, T.x0, T.y0, T.res, 1e6,
                                              0.25))
    edges = int(offsets[-1])
    out["costmap_2048"] = {"ms": ms, "polygons": len(polys), "edges": edges,
                           # most pairs are never evaluated: a tile of nodes
                           # skips the perimeters that cannot touch it
                           "node_edge_pairs_per_s": T.W * T.H * edges * 1e3 / ms,
                           "gb_per_s": 4 * T.W * T.H / ms / 1e6,
                           "hbm_frac": 4 * T.W * T.H / ms / 1e6 / HBM_PEAK_GBS}
    # terrain pack (plan_set_terrain: slopes and the cells' bilinear
    # coefficients, with its non-finite check and the host wait for it):
    # heights and costmap read once, 64-byte cells written
    ms = _time_ms(lambda: pl.set_terrain(h, T.x0, T.y0, T.res, cm))
    nbytes = (4 + 4 + 64) * T.W * T.H
    out["terrain_pack_2048"] = {"ms": ms, "gb_per_s": nbytes / ms / 1e6,
                                "hbm_frac": nbytes / ms / 1e6 / HBM_PEAK_GBS}
    pl.close()
    return out


def serving_leg(scale=1.0, chunk=16, slots=64):
    """Replay the 64-request serving trace (Poisson arrivals at 200 req/s,
    K in {512..8192}, N in 40..160, own 256x256 terrain each) through the
    plain path (one context: set_terrain + rollout + argmin + readback per
    request, FIFO) and through the continuous-batching server. Arrival times
    are multiplied by `scale` (0 = every request arrives at once). Inputs are
    resident on the GPU before the clock starts. Latency = result visible on
    the host minus arrival."""
    import torch
    from paper_2603_20525_amd import inputs
    from paper_2603_20525_amd import plan as P
    reqs = inputs.c3_trace()
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    R = [(r, dev(r.workload.terrain.height), dev(r.workload.controls),
          torch.zeros(r.workload.N, 2, device="cuda")) for r in reqs]
    maxK = max(r.workload.K for r in reqs)
    maxN = max(r.workload.N for r in reqs)
    steps = sum(r.workload.K * r.workload.N * r.workload.integ["substeps"] for r in reqs)
    w0 = reqs[0].workload
    J = torch.empty(maxK, device="cuda")
    pl = P.Planner(w0.vehicle, w0.cost, w0.integ, maxK, maxN, 256, 256)
    srv = P.Server(w0.vehicle, slots, maxK, maxN, 256, 256, 4 << 30, chunk)

    def plain_one(r, h, u, plan):
        w = r.workload
        pl.set_cost(w.cost)
        pl.set_terrain(h, w.terrain.x0, w.terrain.y0, w.terrain.res)
        pl.rollout(w.state0, u, J[:w.K])
        pl.select(u, J[:w.K], plan)

    def submit(r, h, u, plan):
        w = r.workload
        return srv.submit(h, w.terrain.x0, w.terrain.y0, w.terrain.res, w.state0, u, w.cost,
                          w.integ, plan)

    for item in R:  # warm both paths (code objects, first-touch, every slot)
        plain_one(*item)
        submit(*item)
    srv.drain()
    srv.completions(len(R))
    torch.cuda.synchronize()
    # plain path
    lat, done = [], []
    t0 = time.perf_counter() + 0.01
    for r, h, u, plan in R:
        w = r.workload
        arr = t0 + r.arrival * scale
        while time.perf_counter() < arr:
            pass
        plain_one(r, h, u, plan)
        t = time.perf_counter()
        lat.append(t - arr)
        done.append(t)
    plain = _summ(lat, t0, max(done), steps, len(R))
    pl.close()
    # continuous batching
    ts0 = srv.now() + 0.01
    index, lat, done = {}, {}, []
    i = 0
    while len(lat) < len(R):
        now = srv.now()
        while i < len(R) and ts0 + R[i][0].arrival * scale <= now:
            index[submit(*R[i])] = i
            i += 1
        srv.step()
        for rid in srv.completions(len(R)):
            j = index[rid]
            res = srv.result(rid)
            assert res["status"] == 1, res
            lat[j] = res["t_done"] - (ts0 + R[j][0].arrival * scale)
            done.append(res["t_done"])
    serving = _summ(list(lat.values()), ts0, max(done), steps, len(R))
    srv.close()
    return {"plain": plain, "serving": serving}


def measure_plan(w, steps, warmup, lanes=0, block=0, min_latency_plans=100):
    """One workload through the one-launch plan path (rollout + argmin
    epilogue, then the wait for (k*, J*)): the timed region of `steps` plans,
    plan latency over max(steps, min_latency_plans) plans, the kernel's own
    duration from HIP events on the planner's stream, and the two-call path
    (rollout kernel, argmin kernel) for comparison. Inputs are resident in
    HBM before the clock starts."""
    import torch
    from paper_2603_20525_amd import plan as P
    T = w.terrain
    K, N = w.K, w.N
    pl = P.Planner(w.vehicle, w.cost, w.integ, K, N, T.W, T.H)
    pl.set_terrain(torch.from_numpy(T.height).cuda(), T.x0, T.y0, T.res)
    pl.set_launch(lanes, block)
    u = torch.from_numpy(w.controls).cuda()
    J = torch.empty(K, device="cuda")
    plan = torch.empty(N, 2, device="cuda")

    def fused_plan():
        # one launch: rollout + argmin epilogue; the kernel writes (k*, J*)
        # to pinned memory, the call waits for it
        return pl.rollout_argmin(w.state0, u, J, plan)

    def two_call_plan():
        pl.rollout(w.state0, u, J)
        return pl.select(u, J, plan)

    for _ in range(warmup):
        fused_plan()
        two_call_plan()
    torch.cuda.synchronize()

    # timed region: `steps` plans through the one-launch path
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        k_best, j_best = fused_plan()
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0

    # plan latency: each plan from the call to (k*, J*) visible on the host
    n_lat = max(steps, min_latency_plans)
    lat = []
    for _ in range(n_lat):
        ta = time.perf_counter()
        fused_plan()
        lat.append(time.perf_counter() - ta)

    # kernel durations: the library brackets each rollout kernel with HIP
    # events on its own stream (a separate pass, so the timed plans carry no
    # event overhead)
    pl.enable_timing(True)
    kern_ms = []
    for _ in range(n_lat):
        fused_plan()
        kern_ms.append(pl.last_rollout_ms())
    pl.enable_timing(False)

    # the same plans through the two-call path (rollout, then argmin kernel)
    lat2 = []
    torch.cuda.synchronize()
    t2 = time.perf_counter()
    for _ in range(n_lat):
        ta = time.perf_counter()
        r2 = two_call_plan()
        lat2.append(time.perf_counter() - ta)
    torch.cuda.synchronize()
    elapsed2 = time.perf_counter() - t2
    assert r2 == (k_best, j_best), "fused and two-call plans differ"
    lanes_used, block_used = pl.get_launch()
    pl.close()

    steps_per_plan = K * N * w.integ["substeps"]
    k_avg_s = sum(kern_ms) / len(kern_ms) / 1e3
    achieved = OPS_PER_STEP * steps_per_plan / k_avg_s / 1e9
    return {
        "steps_per_plan": steps_per_plan,
        "elapsed_s": elapsed,
        "rollout_steps_per_s": steps_per_plan * steps / elapsed,
        "ms_per_plan": elapsed / steps * 1e3,
        "launch": {"lanes": lanes_used, "block": block_used},
        "plan_latency_ms": {"p50": percentile(lat, 50) * 1e3, "p99": percentile(lat, 99) * 1e3,
                            "plans": n_lat, "path": "one launch + wait for (k*, J*) per plan"},
        "two_call_path": {"rollout_steps_per_s": steps_per_plan * n_lat / elapsed2,
                          "p50_ms": percentile(lat2, 50) * 1e3,
                          "p99_ms": percentile(lat2, 99) * 1e3, "plans": n_lat,
                          "path": "plan_rollout + plan_select(ARGMIN) + wait"},
        "rollout_kernel_ms": {"avg": k_avg_s * 1e3, "min": min(kern_ms), "max": max(kern_ms),
                              "launches": len(kern_ms),
                              "kernel": "rollout_srb (fused argmin epilogue)"},
        "alu_achieved_gops": achieved,
        "best": {"k": k_best, "J": j_best},
    }


def main():
    ap = argparse.ArgumentParser(description=__doc__.split("\n")[0])
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=300)
    ap.add_argument("--warmup", type=int, default=30)
    ap.add_argument("--workload", default="c5", choices=["c2", "c5", "paper"])
    ap.add_argument("--cpu-seconds", type=float, default=10.0,
                    help="seconds of oracle work for cpu_baseline (0 = skip)")
    ap.add_argument("--serving", type=int, default=1,
                    help="also replay the serving trace (plain vs continuous batching)")
    ap.add_argument("--calibrate-copy", type=int, default=0, metavar="MIB",
                    help="only run 5 device-to-device copies of MIB MiB and exit (the "
                         "reference kernel for scaling the HBM byte counters)")
    ap.add_argument("--rows", type=int, default=1,
                    help="also measure the single-plan workload and the widened rows (paper "
                         "shape, EST, RK4, adjoint, terrain preparation)")
    ap.add_argument("--lanes", type=int, default=0)
    ap.add_argument("--block", type=int, default=0)
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py: libplan runs on one GPU; --gpus {args.gpus} is not supported "
              "(sharding candidates over GPUs is designed, not implemented)",
              file=sys.stderr)
        sys.exit(2)

    import torch

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    torch.cuda.set_device(0)
    if args.calibrate_copy:
        n = args.calibrate_copy * (1 << 20) // 4
        src = torch.ones(n, device="cuda")
        dst = torch.empty(n, device="cuda")
        for _ in range(5):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"calibrate_copy_bytes": 4 * n, "copies": 5}), flush=True)
        return
    w, desc = workload(args.workload)
    T = w.terrain
    K, N, S = w.K, w.N, w.integ["substeps"]
    print(f"[bench] workload {args.workload}: {desc}", file=sys.stderr, flush=True)

    m = measure_plan(w, args.steps, args.warmup, args.lanes, args.block)
    print(f"[bench] timed {args.steps} plans in {m['elapsed_s']:.3f} s", file=sys.stderr,
          flush=True)
    achieved = m["alu_achieved_gops"]
    out = {
        "metric": METRIC,
        "value": m["rollout_steps_per_s"],
        "unit": "rollout-steps/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": m["ms_per_plan"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": desc, "K": K, "N": N, "substeps": S, "dt": w.integ["dt"],
                   "terrain": f"{T.W}x{T.H} at {T.res} m", "launch": m["launch"],
                   "path": "plan_rollout_argmin (rollout + argmin in one launch)"},
        "plan_latency_ms": m["plan_latency_ms"],
        "two_call_path": m["two_call_path"],
        "rollout_kernel_ms": m["rollout_kernel_ms"],
        "roofline": {"bound": "alu", "achieved": achieved, "peak": ALU_PEAK_GOPS, "unit": "Gop/s",
                     "frac": achieved / ALU_PEAK_GOPS,
                     "traffic": traffic_bytes(args.workload),
                     "traffic_unit": "bytes per launch (HBM, counter-derived)",
                     "kernel_signature": kernel_signature(),
                     "ops_per_rollout_step": OPS_PER_STEP},
        "best": m["best"],
    }
    if args.rows:
        print("[bench] single-plan workload", file=sys.stderr, flush=True)
        w2, desc2 = workload("c2")
        m2 = measure_plan(w2, args.steps, args.warmup)
        m2.pop("elapsed_s")
        m2["workload"] = desc2
        m2["alu_frac"] = m2.pop("alu_achieved_gops") / ALU_PEAK_GOPS
        m2["traffic"] = traffic_bytes("c2")
        out["single_plan_c2"] = m2
        del w2
    if args.serving:
        print("[bench] serving trace: plain vs continuous batching", file=sys.stderr, flush=True)
        out["serving"] = {
            "trace": "64 requests, Poisson arrivals at 200 req/s, K in {512,1024,2048,4096,8192}, "
                     "N in 40..160, dt 0.02 s, own 256x256 terrain and start each",
            "at_200_req_s": serving_leg(1.0),
            "at_2000_req_s": serving_leg(0.1),
            "burst_all_at_once": serving_leg(0.0),
        }
    if args.rows:
        print("[bench] widened rows", file=sys.stderr, flush=True)
        out["rows"] = rows_leg()
    if args.cpu_seconds > 0:
        print("[bench] timing the FP64 oracle on the host", file=sys.stderr, flush=True)
        out["cpu_baseline"] = cpu_baseline(w, args.cpu_seconds)
    else:
        out["cpu_baseline"] = None
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
