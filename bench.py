"""Benchmark: batched min-cost max-flow on MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--config 4]
    python bench.py --whatif 1        # what-if node addition, paper setting 1
    python bench.py --config 5 --located   # link delays as location latencies
    python bench.py --heuristic        # decentralized heuristic vs the exact optimum

A step solves one whole batch of the workload (every instance to optimality)
with inputs already resident in HBM.  The default workload is the 7B-scale
pipeline batch: 256 instances of 32 stages x 64 nodes with full bipartite
links between consecutive stages (10 locations, supply 512).  Prints one JSON
line: instances solved per second (the value), arc relaxations per second,
the roofline of the solver kernel, and the CPU oracle's rate on a bounded
sample of the same workload.

With --whatif SETTING a step instead evaluates every placement of the
paper's node-addition test (Sec. VI, handling joining nodes; settings 1-3:
8 stages of 12 relays plus one joining position, 8 candidates, 8! = 40320
placements): expand all placements on the device, solve them, reduce to the
best placement.  The value is placements evaluated per second.

With --heuristic a step simulates the paper's decentralized routing
heuristic (Sec. V-C, 120 rounds) on flow-test settings 1-4, 16384 instances
each, and the line scores its cost against the exact optimum of the same
instances (solved on the GPU).  The value is simulated instances per second.

With --located the same preset (2, 4 or 5) is passed in located form (each
node's location and the latency matrix instead of the n x n delays) to
gwtf_mcf_solve_located; the 64 x 512 instance then runs the grid pass with
location-factored relaxation.  That line reports its relaxation operations,
not the dense links they stand for.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0  # MI355X HBM3E, published peak
# Algorithmic bytes of one arc relaxation (examining one residual arc): an
# int32 head, cost and residual, 12 B, as a CSR-streaming solver would read
# them.  The kernel itself streams less (heads implicit, link residuals
# unbounded); the measured HBM traffic is reported beside it.
BYTES_PER_RELAX = 12
# Integer vector peak: 256 CUs x 64 int32 lanes per cycle x 2.4 GHz.  The
# packed pass keeps its link costs in registers and never streams them, so
# its roofline is arithmetic: an add and a min per link relaxation.
ALU_PEAK_TOPS = 256 * 64 * 2.4e9 / 1e12
OPS_PER_RELAX = 2
# VALU issue peak: each CU issues at most one wave64 vector instruction per
# cycle (four SIMDs of 16 lanes, four cycles per wave64 instruction).
VALU_ISSUE_PEAK = 256 * 2.4e9

WORKLOADS = {
    1: "c1: 1024 instances, S=4 x n=4, random costs U[1,100], supply 16",
    2: "c2: 16384 instances, S=8 x n=8, 10-location latencies, supply 64",
    3: "c3: 16384 churn variants of a S=8 x n=8 instance (10-30% nodes deleted, jittered links)",
    4: "c4: 256 instances, S=32 x n=64, full bipartite links, 10-location latencies, supply 512",
    5: "c5: 1 instance, S=64 x n=512, full bipartite links, 10-location latencies, supply 4096",
}


def counter_record(kernel: str, config):
    """The committed rocprofv3 counter record of this kernel on this workload
    (profiles/<kernel>_<workload>_traffic.json), or None when there is none or
    the kernel's sources changed since it was taken."""
    import hashlib

    tag = config if isinstance(config, str) else f"c{config}"
    path = os.path.join(ROOT, "profiles", f"{kernel}_{tag}_traffic.json")
    if not os.path.exists(path):
        return None
    rec = json.load(open(path))
    h = hashlib.sha256()
    for f in rec["sources"]:
        full = os.path.join(ROOT, f)
        if not os.path.exists(full):
            return None
        h.update(open(full, "rb").read())
    return rec if h.hexdigest() == rec["kernel_sources_sha256"] else None


def measured_traffic(kernel: str, config, kernel_s: float):
    """HBM bytes per launch from the committed counter record, as GB/s over
    the measured launch time; None without a current record."""
    rec = counter_record(kernel, config)
    return None if rec is None else rec["traffic_bytes_per_launch"] / kernel_s / 1e9


def valu_issue(kernel: str, config, kernel_s: float):
    """VALU wave-instructions per launch from the committed counter record
    over the measured launch time, against the issue peak (one wave64 vector
    instruction per CU per cycle: four SIMDs of 16 lanes, four cycles each);
    None without a current record with SQ counters."""
    rec = counter_record(kernel, config)
    if rec is None or "sq_counters_per_launch" not in rec:
        return None
    sq = rec["sq_counters_per_launch"]
    achieved = sq["SQ_INSTS_VALU"] / kernel_s
    return {"achieved": achieved, "peak": VALU_ISSUE_PEAK, "unit": "VALU wave-instructions/s",
            "frac": achieved / VALU_ISSUE_PEAK,
            "lds_bank_conflict_cycles_per_lds_instruction": sq["SQ_LDS_BANK_CONFLICT"] / max(1.0, sq["SQ_INSTS_LDS"]),
            "salu_per_cu_cycle": sq["SQ_INSTS_SALU"] / kernel_s / VALU_ISSUE_PEAK,
            "waves": sq["SQ_WAVES"], "counters": f"profiles/{kernel}_{config if isinstance(config, str) else 'c%d' % config}_traffic.json"}


KERNELS = {1: "solve_pipe_kernel", 2: "solve_kernel (LDS state)", 3: "solve_grid_kernel",
           4: "solve_kernel (global-memory state)", 5: "solve_small_kernel (one to sixteen instances per wave)"}
PASS_LAUNCHES = {1: " (keyed launch per step; the unscaled launch after it has no instance and exits)",
                 3: " (one cooperative launch per instance)"}
KERNEL_SYMBOLS = {1: "solve_pipe_kernel", 2: "solve_kernel_lds", 3: "solve_grid_kernel", 4: "solve_kernel_global",
                  5: "solve_small_kernel"}


def cpu_model() -> str:
    """The host CPU's model name from /proc/cpuinfo."""
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def host_threads() -> int:
    threads = int(os.environ.get("OMP_NUM_THREADS", os.cpu_count() or 1))
    return max(1, min(threads, os.cpu_count() or 1))


def oracle_rate(batch, budget_s: float, threads: int):
    """The oracle on `threads` host threads over the batch's instances in
    order, in chunks that grow to about a second each, until `budget_s` is
    spent (starting over when a small batch is done first): (instances done,
    seconds, arc scans, threads used)."""
    import numpy as np

    import oracle
    import oracle.located

    solve = oracle.located.solve if hasattr(batch, "location") else oracle.solve
    done, t_used, scans, used = 0, 0.0, 0, threads
    chunk = max(1, threads)
    while t_used < budget_s:
        first = done % batch.B
        idx = list(range(first, min(batch.B, first + chunk)))
        sub = batch.subset(idx)
        t0 = time.perf_counter()
        r = solve(sub, nthreads=threads, flows=False, potentials=False)
        dt = time.perf_counter() - t0
        t_used += dt
        scans += int(np.sum(r["arc_scans"]))
        done += len(idx)
        used = r["threads"]
        if dt < 0.5:
            chunk = min(4 * chunk, batch.B)
    return done, t_used, scans, used


def cpu_baseline(batch, budget_s: float, threads: int):
    """The oracle on the host cores, on a bounded prefix of the workload:
    all threads for two thirds of the budget, one thread for the rest."""
    done, t_used, scans, used = oracle_rate(batch, budget_s * 2 / 3, threads)
    d1, t1, s1, _ = oracle_rate(batch, budget_s / 3, 1)
    return {"value": done / t_used, "unit": "instances/s", "cores": used, "kind": "oracle",
            "sample": f"{done} instances of the same workload ({batch.B} in the batch, taken in order"
                      f"{', repeated' if done > batch.B else ''}), {t_used:.1f} s wall on {used} threads "
                      f"(one instance per thread)",
            "arc_scans_per_s": scans / t_used,
            "one_core": {"value": d1 / t1, "unit": "instances/s", "arc_scans_per_s": s1 / t1,
                         "sample": f"{d1} instances taken in order, {t1:.1f} s on 1 thread"},
            "cpu_model": cpu_model(), "os_cpu_count": os.cpu_count()}


def cpu_baseline_single(batch, budget_s: float):
    """One huge instance: the oracle solves it on one thread only (its
    shortest-path searches are sequential), so the bounded sample is the same
    instance with the data node's supply capped at A units, i.e. its first A
    augmenting paths; the rate is scaled to the whole instance by its
    augmenting paths (one unit each here: the capped solve finds the same
    first paths).  The time of a complete solve of this instance, stored when
    its optimum was written, is reported beside it."""
    import numpy as np

    import oracle
    import oracle.located

    solve = oracle.located.solve if hasattr(batch, "location") else oracle.solve
    full = json.load(open(os.path.join(ROOT, "tests", "golden", "c5_oracle.json")))
    paths = int(full["augmentations"][0])
    # about 0.25-0.35 s per augmenting path on one core of the test hosts
    units = int(max(8, min(256, budget_s / 0.3)))
    sub = batch.subset([0])
    sub.supply = np.full_like(sub.supply, units)
    t0 = time.perf_counter()
    r = solve(sub, nthreads=1, flows=False, potentials=False)
    t_used = time.perf_counter() - t0
    got = int(r["F"][0])
    est_s = t_used / max(1, got) * paths
    return {"value": 1.0 / est_s, "unit": "instances/s", "cores": 1, "kind": "oracle",
            "sample": f"the same instance with its supply capped at {units} units: {got} augmenting paths "
                      f"in {t_used:.1f} s on 1 thread (graph build included), scaled to the instance's "
                      f"{paths} paths = {est_s:.0f} s per solve",
            "stored_full_solve_s": full["oracle_seconds"], "stored_full_solve_threads": full["oracle_threads"],
            "cpu_model": cpu_model(), "os_cpu_count": os.cpu_count()}


def roofline_for(main_pass, relax, kernel_s, traffic, kernel, issue=None):
    """The packed pass keeps its link costs in registers and issues vector
    instructions back to back: its roofline is the VALU issue rate from the
    committed counters (`issue`), with the two useful integer operations per
    link relaxation (add, min) beside it; without counters, those operations
    against the integer lane peak.  HBM roofline, 12 B per counted
    relaxation, for the passes that stream their arcs.  The stage-pipelined
    passes use latency_roofline instead."""
    if main_pass == 5:
        useful = OPS_PER_RELAX * relax / kernel_s / 1e12
        ops = {"achieved": useful, "peak": ALU_PEAK_TOPS, "unit": "Tops/s", "frac": useful / ALU_PEAK_TOPS,
               "basis": "an add and a min per link relaxation"}
        if issue is not None:
            return {"bound": "alu", "achieved": issue["achieved"], "peak": issue["peak"], "unit": issue["unit"],
                    "frac": issue["frac"], "traffic": traffic, "traffic_unit": "GB/s", "kernel": kernel,
                    "kernel_ms": kernel_s * 1e3, "issue": issue, "useful_ops": ops}
        return {"bound": "alu", "achieved": useful, "peak": ALU_PEAK_TOPS, "unit": "Tops/s",
                "frac": useful / ALU_PEAK_TOPS, "traffic": traffic, "traffic_unit": "GB/s",
                "kernel": kernel, "kernel_ms": kernel_s * 1e3}
    counted = BYTES_PER_RELAX * relax / kernel_s / 1e9
    return {"bound": "hbm", "achieved": counted, "peak": HBM_PEAK_GBS, "unit": "GB/s",
            "frac": counted / HBM_PEAK_GBS, "traffic": traffic, "kernel": kernel, "kernel_ms": kernel_s * 1e3}


def pipeline_depth(main_pass, S):
    """Owners a label passes through in the first iteration of a search:
    the register pass gives each wave two stages above 16 stages (one
    below), the grid pass one stage per group of workgroups."""
    if main_pass == 1:
        return -(-S // (2 if S > 16 else 1))
    return S


def latency_roofline(main_pass, stats, S, kernel_s, handoff, traffic, kernel):
    """Critical-path model of the stage-pipelined passes.  Iteration t of a
    search at pipeline position k waits for position k-1 at iteration t and
    position k+1 at iteration t-1, so a search that converges at iteration
    T_s costs (H - 1) + 2 (T_s - 1) sequential hand-offs, H the pipeline
    depth.  The unit is such a hop; the floor of one hop is the bare hand-off
    latency measured on this device in the same run (LDS between two waves
    for the register pass, device-scope between neighbouring stages'
    workgroups for the grid pass).  achieved = hops on the launch's critical
    path / kernel time (the batch's slowest instance for the register pass,
    which solves one instance per workgroup); frac = that time floor / the
    measured time."""
    import numpy as np

    H = pipeline_depth(main_pass, S)
    rounds = stats[:, 1].astype(np.float64)
    searches = (stats[:, 8] if main_pass == 3 else stats[:, 0]).astype(np.float64)
    hops = searches * (H - 1) + 2.0 * (rounds - searches)
    crit = float(hops.max())
    floor_ns = handoff["lds_wave_ns"] if main_pass == 1 else handoff["device_neighbour_ns"]
    if floor_ns <= 0:
        return {"bound": "latency", "achieved": None, "peak": None, "frac": None, "traffic": traffic,
                "kernel": kernel, "kernel_ms": kernel_s * 1e3, "note": "hand-off calibration failed"}
    achieved = crit / kernel_s
    peak = 1e9 / floor_ns
    return {"bound": "latency", "achieved": achieved, "peak": peak, "unit": "pipeline hops/s",
            "frac": achieved / peak, "traffic": traffic, "traffic_unit": "GB/s", "kernel": kernel,
            "kernel_ms": kernel_s * 1e3,
            "model": {"pipeline_depth": H, "searches": float(searches[int(hops.argmax())]),
                      "iterations": float(rounds[int(hops.argmax())]), "critical_hops": crit,
                      "hop_floor_ns": floor_ns,
                      "hop_floor": "LDS wave-to-wave hand-off" if main_pass == 1
                      else "device-scope hand-off between neighbouring stages' workgroups",
                      "ns_per_hop": kernel_s * 1e9 / crit, "handoff_calibration_ns": handoff}}


def heuristic_counters():
    """Per-setting counters of the heuristic kernel from the committed
    rocprofv3 record, or None when the kernel's sources changed since."""
    import hashlib

    path = os.path.join(ROOT, "profiles", "heuristic_kernel_flowtests_counters.json")
    if not os.path.exists(path):
        return None
    rec = json.load(open(path))
    h = hashlib.sha256()
    for f in rec["sources"]:
        full = os.path.join(ROOT, f)
        if not os.path.exists(full):
            return None
        h.update(open(full, "rb").read())
    return rec if h.hexdigest() == rec["kernel_sources_sha256"] else None


def heuristic_roofline(instance_rounds, kernel_ms, batch):
    """The heuristic simulation keeps each instance in LDS and issues vector
    instructions back to back.  Its roofline is that issue rate: VALU
    wave-instructions per launch (the committed counter record, which holds
    for the same sources, batch and seed) over the measured kernel time."""
    rec = heuristic_counters()
    total_s = sum(kernel_ms.values()) / 1e3
    line = {"bound": "alu", "unit": "VALU wave-instructions/s", "peak": VALU_ISSUE_PEAK,
            "achieved": None, "frac": None, "traffic": None,
            "kernel": "heuristic_kernel (one launch per setting, heuristic_general_kernel after it)", "kernel_ms": total_s * 1e3,
            "instance_rounds_per_s": instance_rounds / total_s}
    if rec is not None and batch == 16384:
        per = rec["per_setting"]
        valu = sum(per[f"setting {s}"]["SQ_INSTS_VALU"] for s in kernel_ms)
        traffic = sum(per[f"setting {s}"]["traffic_bytes"] for s in kernel_ms)
        line.update(achieved=valu / total_s, frac=valu / total_s / VALU_ISSUE_PEAK,
                    traffic=traffic / total_s / 1e9, traffic_unit="GB/s",
                    valu_per_instance_round=valu / instance_rounds,
                    counters="profiles/heuristic_kernel_flowtests_counters.json")
    return line


def whatif_cpu_baseline(base, slot, cands, total: int, budget_s: float, threads: int):
    """The oracle (expansion and solve) on the host cores, on a bounded prefix
    of the placements."""
    import oracle
    import oracle.whatif as OW

    done, t_used, chunk = 0, 0.0, 256
    while done < total and t_used < budget_s:
        cnt = min(chunk, total - done)
        t0 = time.perf_counter()
        batch = OW.expand(base, slot, cands, done, cnt)
        r = oracle.solve(batch, nthreads=threads, flows=False, potentials=False)
        t_used += time.perf_counter() - t0
        done += cnt
        used = r["threads"]
    return {"value": done / t_used, "unit": "placements/s", "cores": used, "kind": "oracle",
            "sample": f"first {done} of {total} placements of the same problem, expanded and solved, "
                      f"{t_used:.1f} s wall on {used} threads"}


def run_whatif(args):
    """Time whole what-if evaluations: expand + solve + best placement."""
    import numpy as np
    import torch

    from paper_2509_21221_amd import workloads as W
    from paper_2509_21221_amd.mcf import Solver, gwtf_whatif_count

    base, slot, cands = W.node_addition(args.whatif)
    S, n = base.S, base.n
    total = gwtf_whatif_count(S, cands.m)
    dev = torch.device("cuda", 0)
    torch.cuda.set_device(dev)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    bt = {"node_cap": t(base.node_cap), "node_cost": t(base.node_cost), "arc_cost": t(base.arc_cost),
          "src_cost": t(base.src_cost), "snk_cost": t(base.snk_cost), "supply": t(base.supply)}
    ct = {"cap": t(cands.cap), "cost": t(cands.cost), "in_cost": t(cands.inn), "out_cost": t(cands.out),
          "link_cost": t(cands.link), "src_cost": t(cands.src), "snk_cost": t(cands.snk)}
    stream = torch.cuda.current_stream(dev)
    solver = Solver(S, n, total, device=0, stream=stream)
    e = lambda *shape, dt=torch.int32: torch.empty(shape, dtype=dt, device=dev)
    batch = {"node_cap": e(total, S, n), "node_cost": e(total, S, n), "arc_cost": e(total, S - 1, n, n),
             "src_cost": e(total, n), "snk_cost": e(total, n), "supply": e(total)}
    outs = (e(total, dt=torch.int64), e(total, dt=torch.int64), e(total))
    best = e(3, dt=torch.int64)

    def step():
        solver.whatif_expand(bt, ct, slot, 0, total, out=batch)
        solver.solve(batch["node_cap"], batch["node_cost"], batch["arc_cost"], batch["supply"],
                     src_cost=batch["src_cost"], snk_cost=batch["snk_cost"], out=outs)
        solver.whatif_best(*outs, first=0, best=best)

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    # phase split of one evaluation, on the solver's stream
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
    ev[0].record(stream)
    solver.whatif_expand(bt, ct, slot, 0, total, out=batch)
    ev[1].record(stream)
    solver.solve(batch["node_cap"], batch["node_cost"], batch["arc_cost"], batch["supply"],
                 src_cost=batch["src_cost"], snk_cost=batch["snk_cost"], out=outs)
    ev[2].record(stream)
    solver.whatif_best(*outs, first=0, best=best)
    ev[3].record(stream)
    torch.cuda.synchronize()
    expand_ms, solve_ms, best_ms = (ev[i].elapsed_time(ev[i + 1]) for i in range(3))

    starts = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps)]
    ends = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps)]
    t0 = time.perf_counter()
    for k in range(args.steps):
        starts[k].record(stream)
        step()
        ends[k].record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    status = outs[2].cpu().numpy()
    if (status != 0).any():
        raise SystemExit(f"solver reported non-ok status on {(status != 0).sum()} placements")
    stats = solver.stats().cpu().numpy()
    passes = solver.passes().cpu().numpy()
    main_pass = int(np.bincount(passes).argmax())
    relax = int(stats[:, 2].sum()) * n + int(stats[:, 3].sum())
    solve_s = solve_ms / 1e3
    b = best.cpu().numpy()
    inst_ints = 2 * S * n + (S - 1) * n * n + 2 * n + 1
    line = {
        "metric": "what-if placements evaluated/sec (expand + solve + best placement)",
        "value": total * args.steps / wall,
        "unit": "placements/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": wall / args.steps * 1e3,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "int32", "data": "synthetic (seeded generator, paper-shaped)",
        "config": {"workload": f"node addition setting {args.whatif}: S={S} x n={n} ({n - 1} relays + 1 "
                               f"joining position), {cands.m} candidates, {total} placements, supply "
                               f"{int(base.supply[0])}", "placements": total, "stages": S,
                   "nodes_per_stage": n, "seed": 0},
        "best_placement": {"index": int(b[0]), "F": int(b[1]), "cost": int(b[2])},
        "phase_ms": {"expand": expand_ms, "solve": solve_ms, "best": best_ms},
        "expand_write_GBs": 4 * inst_ints * total / (expand_ms / 1e3) / 1e9,
        "arc_relaxations_per_s": relax / solve_s,
        "roofline": roofline_for(main_pass, relax, solve_s,
                                 measured_traffic(KERNEL_SYMBOLS.get(main_pass, "?"), f"whatif{args.whatif}", solve_s),
                                 KERNELS.get(main_pass, "?") + " (one launch per step)",
                                 valu_issue(KERNEL_SYMBOLS.get(main_pass, "?"), f"whatif{args.whatif}", solve_s)),
    }
    if args.cpu_budget > 0:
        threads = int(os.environ.get("OMP_NUM_THREADS", os.cpu_count() or 1))
        threads = max(1, min(threads, os.cpu_count() or 1))
        line["cpu_baseline"] = whatif_cpu_baseline(base, slot, cands, total, args.cpu_budget, threads)
    solver.close()
    print(json.dumps(line), flush=True)


def run_churn(args):
    """Time warm-started re-solves of the churn variants of the 8 x 8 base
    instance from the base's optimal flow, beside cold solves of the same
    batch."""
    import numpy as np
    import torch

    from paper_2509_21221_amd import workloads as W
    from paper_2509_21221_amd.mcf import Solver

    base, var = W.config2(1, 0), W.config3(16384, 0)
    S, n, B = var.S, var.n, var.B
    dev = torch.device("cuda", 0)
    torch.cuda.set_device(dev)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    stream = torch.cuda.current_stream(dev)
    with Solver(S, n, 1, device=0, stream=stream) as s0:
        s0.solve(t(base.node_cap), t(base.node_cost), t(base.arc_cost), t(base.supply),
                 t(base.src_cost), t(base.snk_cost))
        start = {k: v[:1].clone() for k, v in s0.flows().items() if k != "potential"}
    solver = Solver(S, n, B, device=0, stream=stream)
    args_v = (t(var.node_cap), t(var.node_cost), t(var.arc_cost), t(var.supply))
    costs = dict(src_cost=t(var.src_cost), snk_cost=t(var.snk_cost))
    warm = lambda: solver.resolve_churn(*args_v, start, **costs)
    cold = lambda: solver.solve(*args_v, **costs)
    for _ in range(args.warmup):
        warm()
        cold()
    torch.cuda.synchronize()

    def timed(fn):
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        ev[0].record(stream)
        for _ in range(args.steps):
            out = fn()
        ev[1].record(stream)
        torch.cuda.synchronize()
        return ev[0].elapsed_time(ev[1]) / args.steps, out

    t0 = time.perf_counter()
    warm_ms, (Fw, Cw, Sw) = timed(warm)
    wall = time.perf_counter() - t0
    cold_ms, (Fc, Cc, Sc) = timed(cold)
    Fw, Cw, Sw, Fc, Cc, Sc = (x.cpu().numpy() for x in (Fw, Cw, Sw, Fc, Cc, Sc))
    if (Sw != 0).any() or not ((Fw == Fc).all() and (Cw == Cc).all()):
        raise SystemExit("warm-started and cold solves disagree")
    _, _, _, wk = solver.resolve_churn(*args_v, start, **costs, work=True)
    wk = wk.cpu().numpy()
    passes = solver.passes().cpu().numpy()
    # The kernel is a chain of label-correcting rounds per instance, several
    # instances per wave: bound by the dependent instructions of a round, not
    # by memory (its inputs are read once: inst_bytes per instance).
    inst_bytes = 4 * (2 * S * n + (S - 1) * n * n + 2 * n + 1) + 20
    rounds_total = float(wk[:, 3].sum())
    line = {
        "metric": "churn variants re-solved/sec (warm start from the base optimum)",
        "value": B / (warm_ms / 1e3),
        "unit": "instances/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": wall / args.steps * 1e3,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "int32", "data": "synthetic (seeded generator, paper-shaped)",
        "config": {"workload": f"{B} churn variants of one S={S} x n={n} instance (10-30 % of nodes "
                               "deleted, delays jittered), start = the base's optimal flow",
                   "instances": B, "stages": S, "nodes_per_stage": n, "seed": 0},
        "cold_solve_ms": cold_ms, "cold_pass": int(np.bincount(passes).argmax()),
        "warm_ms": warm_ms,
        "work_mean": {"paths_removed": float(wk[:, 0].mean()), "cycles_cancelled": float(wk[:, 1].mean()),
                      "augmentations": float(wk[:, 2].mean()), "rounds": float(wk[:, 3].mean())},
        "roofline": {"bound": "latency", "achieved": rounds_total / (warm_ms / 1e3),
                     "unit": "label-correcting rounds/s (all instances)", "peak": None, "frac": None,
                     "traffic": inst_bytes * B / (warm_ms / 1e3) / 1e9, "traffic_unit": "GB/s (inputs read once)",
                     "kernel": "churn_packed_kernel (churn_kernel after it for what it passes on)",
                     "note": "the cold packed pass needs fewer label-correcting passes on this workload "
                             "(cold_solve_ms)"},
    }
    if args.cpu_budget > 0:
        line["cpu_baseline"] = cpu_baseline(var, args.cpu_budget, host_threads())
    solver.close()
    print(json.dumps(line), flush=True)


def run_heuristic(args):
    """Time the decentralized-heuristic simulation on flow-test settings 1-4
    and score it against the exact optimum of the same instances."""
    import numpy as np
    import torch

    from paper_2509_21221_amd import workloads as W
    from paper_2509_21221_amd.mcf import Solver

    dev = torch.device("cuda", 0)
    torch.cuda.set_device(dev)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    stream = torch.cuda.current_stream(dev)
    B, rounds, settings = args.heuristic_batch, args.rounds, (1, 2, 3, 4)
    jobs = []
    for s in settings:
        batch = W.paper_flow_test(s, B)
        solver = Solver(batch.S, batch.n, B, device=0, stream=stream)
        inputs = (t(batch.node_cap), t(batch.node_cost), t(batch.arc_cost), t(batch.supply),
                  t(batch.src_cost), t(batch.snk_cost))
        # slots (LDS) sized to the batch's largest total capacity
        slots = int(-(-int(batch.node_cap.sum(axis=(1, 2)).max()) // 32) * 32)
        jobs.append((s, batch, solver, inputs, slots))

    def step():
        return [solver.simulate_heuristic(*inp, rounds=rounds, objective=args.objective, seed=0,
                                          max_slots=slots) for _, _, solver, inp, slots in jobs]

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in jobs]
    t0 = time.perf_counter()
    for k in range(args.steps):
        for (s, batch, solver, inp, slots), (e0, e1) in zip(jobs, ev):
            if k == args.steps - 1:
                e0.record(stream)
            solver.simulate_heuristic(*inp, rounds=rounds, objective=args.objective, seed=0, max_slots=slots)
            if k == args.steps - 1:
                e1.record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    kernel_ms = {s: e0.elapsed_time(e1) for (s, *_), (e0, e1) in zip(jobs, ev)}
    per_setting = {}
    for s, batch, solver, inp, slots in jobs:
        F, cost, status = (x.cpu().numpy() for x in solver.simulate_heuristic(
            *inp, rounds=rounds, objective=args.objective, seed=0, max_slots=slots))
        eF, ecost, estatus = (x.cpu().numpy() for x in solver.solve(*inp[:4], src_cost=inp[4], snk_cost=inp[5]))
        if (status != 0).any() or (estatus != 0).any():
            raise SystemExit(f"setting {s}: non-ok status")
        same = F == eF
        per_setting[f"setting {s}"] = {
            "stages": batch.S, "relays_per_stage": batch.n,
            "heuristic_over_optimum": float(cost[same].sum() / ecost[same].sum()),
            "mean_instance_ratio": float(np.mean(cost[same] / ecost[same])),
            "reached_optimal_flow": float(same.mean()),
            "max_slots": slots, "kernel_ms": kernel_ms[s]}
    total_ms = sum(kernel_ms.values())
    line = {
        "metric": "decentralized-heuristic instances simulated/sec (120 rounds) and cost / exact optimum",
        "value": len(jobs) * B * args.steps / wall,
        "unit": "instances/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": wall / args.steps * 1e3,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "int32+f64", "data": "synthetic (seeded generator, paper-shaped)",
        "config": {"workload": f"flow-test settings 1-4 (40 relays over 8 or 10 stages, one data node), {B} "
                               f"instances each, {rounds} rounds, {args.objective} objective, T0 1.7, alpha 0.95",
                   "instances": len(jobs) * B, "rounds": rounds, "seed": 0},
        "instance_rounds_per_s": len(jobs) * B * rounds / (total_ms / 1e3),
        "per_setting": per_setting,
        # the committed counters hold for the default workload only
        "roofline": heuristic_roofline(len(jobs) * B * rounds, kernel_ms,
                                       B if (args.objective, rounds) == ("sum", 120) else 0),
    }
    if args.cpu_budget > 0:
        from oracle import heuristic as H

        threads = int(os.environ.get("OMP_NUM_THREADS", os.cpu_count() or 1))
        threads = max(1, min(threads, os.cpu_count() or 1))
        done, used_s = 0, 0.0
        while used_s < args.cpu_budget and done < B:
            for s, batch, *_ in jobs:
                sub = batch.subset(range(done, min(B, done + 256)))
                t1 = time.perf_counter()
                r = H.simulate(sub, rounds=rounds, objective=args.objective, seed=0, nthreads=threads)
                used_s += time.perf_counter() - t1
            done = min(B, done + 256)
        line["cpu_baseline"] = {"value": len(jobs) * done / used_s, "unit": "instances/s", "cores": r["threads"],
                                "kind": "oracle",
                                "sample": f"first {done} instances of each of the 4 settings, {used_s:.1f} s wall "
                                          f"on {r['threads']} threads"}
    for _, _, solver, _, _ in jobs:
        solver.close()
    print(json.dumps(line), flush=True)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--config", type=int, default=4, choices=sorted(WORKLOADS))
    ap.add_argument("--whatif", type=int, default=0, choices=[0, 1, 2, 3],
                    help="time what-if node addition for this paper setting instead (0 = off)")
    ap.add_argument("--churn", action="store_true",
                    help="warm-started re-solve of the 8x8 churn variants beside cold solves")
    ap.add_argument("--heuristic", action="store_true",
                    help="simulate the decentralized heuristic on flow-test settings 1-4 and score it")
    ap.add_argument("--heuristic-batch", type=int, default=16384, help="instances per setting (--heuristic)")
    ap.add_argument("--rounds", type=int, default=120, help="heuristic rounds (--heuristic)")
    ap.add_argument("--objective", choices=["sum", "max"], default="sum", help="heuristic objective")
    ap.add_argument("--located", action="store_true",
                    help="pass the preset (2, 4 or 5) in located form to gwtf_mcf_solve_located")
    ap.add_argument("--cpu-budget", type=float, default=15.0,
                    help="seconds of oracle time for the CPU baseline (0 = skip)")
    ap.add_argument("--calibrate-copy", type=int, default=0, metavar="MIB",
                    help="only run one device-to-device copy of MIB MiB (counter calibration)")
    args = ap.parse_args()
    if args.calibrate_copy:
        import torch

        nbytes = args.calibrate_copy << 20
        src = torch.ones(nbytes // 4, dtype=torch.int32, device="cuda")
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"copy_bytes_read": nbytes, "copy_bytes_written": nbytes}), flush=True)
        return
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only: this solver has no multi-GPU path "
              f"(--gpus {args.gpus} requested)", file=sys.stderr)
        sys.exit(2)

    if args.whatif:
        return run_whatif(args)
    if args.churn:
        return run_churn(args)
    if args.heuristic:
        return run_heuristic(args)

    import numpy as np
    import torch

    from paper_2509_21221_amd import workloads as W
    from paper_2509_21221_amd.mcf import Solver

    if args.located and args.config not in (2, 4, 5):
        raise SystemExit("--located applies to the location-latency presets 2, 4 and 5")
    batch = W.located(args.config) if args.located else W.CONFIGS[args.config]()
    dev = torch.device("cuda", 0)
    torch.cuda.set_device(dev)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    if args.located:
        inputs = (t(batch.node_cap), t(batch.node_cost), t(batch.location), t(batch.latency),
                  t(batch.supply), t(batch.src_cost), t(batch.snk_cost))
    else:
        inputs = (t(batch.node_cap), t(batch.node_cost), t(batch.arc_cost) if batch.S > 1 else None,
                  t(batch.supply), t(batch.src_cost), t(batch.snk_cost))
    stream = torch.cuda.current_stream(dev)
    solver = Solver(batch.S, batch.n, batch.B, device=0, stream=stream)
    outs = (torch.empty(batch.B, dtype=torch.int64, device=dev),
            torch.empty(batch.B, dtype=torch.int64, device=dev),
            torch.empty(batch.B, dtype=torch.int32, device=dev))

    def step():
        if args.located:
            solver.solve_located(*inputs[:5], src_cost=inputs[5], snk_cost=inputs[6], out=outs)
        else:
            solver.solve(*inputs[:4], src_cost=inputs[4], snk_cost=inputs[5], out=outs)

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    starts = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps)]
    ends = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps)]
    t0 = time.perf_counter()
    for k in range(args.steps):
        starts[k].record(stream)
        step()
        ends[k].record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    ev_ms = [s.elapsed_time(e) for s, e in zip(starts, ends)]

    status = outs[2].cpu().numpy()
    if (status != 0).any():
        raise SystemExit(f"solver reported non-ok status on {(status != 0).sum()} instances")
    stats = solver.stats().cpu().numpy()
    passes = solver.passes().cpu().numpy()
    main_pass = int(np.bincount(passes).argmax())
    rows, pulls = int(stats[:, 2].sum()), int(stats[:, 3].sum())
    dense_relax = rows * batch.n
    relax = dense_relax + pulls
    kernel_s = float(np.mean(ev_ms)) / 1e3
    S_, n_ = batch.S, batch.n
    res_arcs = 2 * (1 + 2 * n_ + S_ * n_ + (S_ - 1) * n_ * n_)  # residual arcs, every link present
    floor_bytes = BYTES_PER_RELAX * res_arcs * float(stats[:, 0].sum())
    floor_gbs = floor_bytes / kernel_s / 1e9
    kernel = KERNELS.get(main_pass, "?") + PASS_LAUNCHES.get(main_pass, " (one launch per step)")
    traffic = measured_traffic(KERNEL_SYMBOLS.get(main_pass, "?"),
                               f"c{args.config}_located" if args.located else args.config, kernel_s)
    if main_pass in (1, 3):
        # stage-pipelined passes: link costs stay on chip, the hand-offs
        # between stages bound them
        from paper_2509_21221_amd.mcf import gwtf_mcf_calibrate_handoff

        handoff = gwtf_mcf_calibrate_handoff(0, stream.cuda_stream, max(1, -(-batch.n // 128)) if main_pass == 3
                                             else 4)
        roof = latency_roofline(main_pass, stats, batch.S, kernel_s, handoff, traffic, kernel)
        roof["issue"] = valu_issue(KERNEL_SYMBOLS.get(main_pass, "?"),
                                   f"c{args.config}_located" if args.located else args.config, kernel_s)
        if not args.located:
            # The 12 B per residual arc of a sweep-based method, one sweep per
            # augmenting path, over the same time: what a CSR-streaming
            # solver would need from HBM to match this speed.
            counted = BYTES_PER_RELAX * relax / kernel_s / 1e9
            roof["hbm_floor_equivalent"] = {
                "achieved": floor_gbs, "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": floor_gbs / HBM_PEAK_GBS,
                "bytes_per_launch": floor_bytes,
                "basis": "12 B x residual arcs x augmenting paths (one sweep per path)",
                "counted_work": {"achieved": counted, "frac": counted / HBM_PEAK_GBS, "unit": "GB/s",
                                 "basis": "12 B per relaxation performed; link costs stay on chip"}}
    else:
        roof = roofline_for(main_pass, relax, kernel_s, traffic, kernel,
                            valu_issue(KERNEL_SYMBOLS.get(main_pass, "?"),
                                       f"c{args.config}_located" if args.located else args.config, kernel_s))
        # The same 12 B per residual arc at the floor of a sweep-based
        # method: one pass over every residual arc per augmenting path.
        roof["sweep_floor"] = {"achieved": floor_gbs, "frac": floor_gbs / HBM_PEAK_GBS,
                               "unit": "GB/s", "bytes": floor_bytes}
    roof["instances_per_pass"] = {KERNELS[p]: int((passes == p).sum()) for p in np.unique(passes)}

    line = {
        "metric": "MCMF instances solved/sec (+ arc relaxations/sec, % of HBM roofline)",
        "value": batch.B * args.steps / wall,
        "unit": "instances/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": wall / args.steps * 1e3,
        "ms_per_step_median": float(np.median(ev_ms)),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "int32", "data": "synthetic (seeded generator, paper-shaped)",
        "config": {"workload": WORKLOADS[args.config] + (", located form (node locations + latency matrix)"
                                                          if args.located else ""),
                   "instances": batch.B, "stages": batch.S, "nodes_per_stage": batch.n, "seed": 0},
        "arc_relaxations_per_s": relax / kernel_s,
        "dense_link_relaxations_per_s": dense_relax / kernel_s,
        "augmentations_per_instance": float(stats[:, 0].mean()),
        "rounds_per_augmentation": float(stats[:, 1].sum() / max(1, stats[:, 0].sum())),
        "phase_ms_per_instance": {name: float(stats[:, col].mean()) / 1e6 for name, col in
                                  (("forward", 4), ("backward", 5), ("augment", 6), ("other", 7))},
        "roofline": roof,
    }
    if main_pass == 3:
        line["searches_per_instance"] = float(stats[:, 8].mean())
        line["phase_ms_per_instance"] = {name: float(stats[:, col].mean()) / 1e6 for name, col in
                                         (("label_iterations", 4), ("potentials_walks_augment", 6),
                                          ("resets_barriers", 7))}
    else:
        line["layer_steps_per_augmentation"] = {
            "forward": float(stats[:, 8].sum() / max(1, stats[:, 0].sum())),
            "backward": float(stats[:, 9].sum() / max(1, stats[:, 0].sum()))}
    if args.located:
        line["metric"] = "MCMF instances solved/sec, located form (+ relaxation operations/sec)"
        line["factored_relaxation_ops_per_s"] = relax / kernel_s if main_pass == 3 else None
        line["arc_relaxations_per_s"] = None if main_pass == 3 else line["arc_relaxations_per_s"]
        line["dense_link_relaxations_per_s"] = None
    if args.cpu_budget > 0 and batch.B == 1:
        line["cpu_baseline"] = cpu_baseline_single(batch, args.cpu_budget)
    elif args.cpu_budget > 0:
        line["cpu_baseline"] = cpu_baseline(batch, args.cpu_budget, host_threads())
    solver.close()
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
