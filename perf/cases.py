"""The calls whose speed this repository is judged by: what a program that
routes microbatches with it asks of it, through ``mcf.Solver``.

Kinds:

* ``solve``: exact min-cost max-flow of a batch, dense link delays;
* ``located``: the same for instances given by locations and latencies;
* ``churn``: warm-started re-solve of churned variants of one base pipeline
  from the base's optimal flow;
* ``whatif``: node addition, one call chain of expand, solve and best;
* ``heuristic``: simulation of the decentralized protocol.

Recipes of the ``solve`` instances: ``uniform`` (capacities U[1, cap_hi],
node and link costs U[1, cost_hi]; a share ``holes`` of the links missing and
a share ``dead`` of the nodes gone), ``geo`` (nodes at 10 locations, link
delay = latency of the two locations, lognormal compute costs), ``flow`` (the
paper's flow-test table: 40 relays, link costs only, the data node's supply
equal to the relays' total capacity).

Optimal flows are not unique (equal delays are common), so the outputs are
the value, the cost and the status of every instance, which are; reading a
flow back is a device copy.  The heuristic's result is unique (its random
numbers are counter-based), and all of it is returned.
"""
import math

import numpy as np
import torch

from paper_2509_21221_amd.mcf import Solver

LOCATIONS = 10
# stages, nodes, capacity range, link-cost range of the paper's flow tests
FLOW_TESTS = {1: (8, 5, (1, 3), (1, 20)), 2: (10, 4, (1, 3), (1, 20)),
              3: (8, 5, (5, 15), (1, 20)), 4: (8, 5, (1, 3), (5, 100))}
# stages, capacity range, link-cost range of the paper's node-addition tests
NODE_TESTS = {1: (8, (1, 20), (1, 100)), 2: (8, (1, 20), (20, 100)),
              3: (8, (1, 5), (1, 100)), 4: (12, (1, 20), (1, 100))}


def _solve(stages, nodes, batch, recipe, cap_hi, cost_hi, supply, holes=0.0, dead=0.0):
    return {"kind": "solve", "stages": stages, "nodes": nodes, "batch": batch, "recipe": recipe,
            "cap_hi": cap_hi, "cost_hi": cost_hi, "supply": supply, "holes": holes, "dead": dead}


def _flow_test(setting, batch):
    S, n, (_, cap_hi), (_, cost_hi) = FLOW_TESTS[setting]
    return dict(_solve(S, n, batch, "flow", cap_hi, cost_hi, -1), setting=setting)


def _located(stages, nodes, batch, cap_hi, supply):
    return {"kind": "located", "stages": stages, "nodes": nodes, "batch": batch, "cap_hi": cap_hi, "supply": supply}


def _churn(stages, nodes, batch, cap_hi, supply):
    return {"kind": "churn", "stages": stages, "nodes": nodes, "batch": batch, "cap_hi": cap_hi, "supply": supply}


def _whatif(setting, first, count):
    return {"kind": "whatif", "setting": setting, "first": first, "count": count, "supply": 64}


def _heuristic(setting, batch, rounds, objective):
    return {"kind": "heuristic", "setting": setting, "batch": batch, "rounds": rounds, "objective": objective}


def listed():
    return [
        # one data node routes its pipeline when a node joins or leaves: the
        # smallest call, launches and one instance's chain of searches
        dict(_solve(8, 8, 1, "geo", 8, 0, 64), name="one_8x8"),
        # a small batch of tiny pipelines (the repository's first preset)
        dict(_solve(4, 4, 1024, "uniform", 4, 100, 16), name="batch_4x4"),
        # a large batch of the paper-shaped pipeline (second preset)
        dict(_solve(8, 8, 16384, "geo", 8, 0, 64), name="batch_8x8_geo"),
        # optimum that the flow ablation scores the heuristic against:
        # capacities 5 to 14, so the supply is several hundred microbatches
        dict(_flow_test(3, 4096), name="flow_test_3"),
        # delays in finer units (up to 6000), links and nodes missing, odd sizes
        dict(_solve(7, 11, 1500, "uniform", 6, 6000, 60, 0.1, 0.05), name="fine_delays_7x11"),
        # every placement of joining nodes, 8 stages (40,320 instances)
        dict(_whatif(1, 0, 40320), name="join_8_stages"),
        # one chunk of the 12! placements of the 12-stage setting
        dict(_whatif(4, 1000003, 8192), name="join_12_stages"),
        # warm-started re-solve of churned variants (third preset's churn)
        dict(_churn(8, 8, 16384, 8, 64), name="churn_8x8"),
        # the protocol's simulation in the flow ablation
        dict(_heuristic(1, 16384, 120, "sum"), name="heuristic_1"),
        # the headline batch: 256 pipelines of 32 stages x 64 nodes
        dict(_solve(32, 64, 256, "geo", 8, 0, 512), name="batch_32x64_geo"),
        # wide stages given by location, a few at once, ragged width
        dict(_located(16, 200, 4, 8, 400), name="located_16x200"),
        # the single huge pipeline (fifth preset)
        dict(_solve(64, 512, 1, "geo", 16, 0, 4096), name="one_64x512_geo"),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def draw(rng):
    kind = rng.choice(["small", "small", "small_fine", "flow", "deep", "join", "churn", "heuristic", "pipeline",
                       "pipeline", "wide"])
    if kind == "small":
        S, n = rng.randint(2, 8), rng.randint(2, 16)
        if rng.random() < 0.5:
            return _solve(S, n, _log(rng, 1, 16384), "geo", rng.randint(2, 8), 0, rng.randint(8, 100))
        return _solve(S, n, _log(rng, 1, 16384), "uniform", rng.randint(2, 8), rng.randint(20, 2000),
                      rng.randint(8, 100), rng.choice([0.0, 0.1]), rng.choice([0.0, 0.1]))
    if kind == "small_fine":
        return _solve(rng.randint(2, 8), rng.randint(3, 16), _log(rng, 16, 2048), "uniform", rng.randint(2, 8),
                      rng.randint(2100, 60000), rng.randint(8, 100), rng.choice([0.0, 0.1]), rng.choice([0.0, 0.1]))
    if kind == "flow":
        return _flow_test(rng.randint(1, 4), _log(rng, 64, 6000))
    if kind == "deep":
        S, n = rng.randint(9, 16), rng.randint(3, 16)
        recipe, cost_hi = rng.choice([("geo", 0), ("uniform", 500)])
        return _solve(S, n, _log(rng, 16, 4096), recipe, rng.randint(2, 8), cost_hi, rng.randint(8, 100))
    if kind == "join":
        setting = rng.randint(1, 4)
        S = NODE_TESTS[setting][0]
        count = _log(rng, 500, 40320 if S == 8 else 8192)
        return _whatif(setting, rng.randint(0, math.factorial(S) - count), count)
    if kind == "churn":
        return _churn(rng.randint(4, 8), rng.randint(4, 10), _log(rng, 256, 8192), rng.randint(2, 8),
                      rng.randint(16, 64))
    if kind == "heuristic":
        return _heuristic(rng.randint(1, 4), _log(rng, 256, 16384), rng.randint(30, 120), rng.choice(["sum", "max"]))
    if kind == "pipeline":
        S, n, B = rng.randint(4, 32), rng.randint(17, 64), _log(rng, 4, 256)
        if rng.random() < 0.5:
            return _solve(S, n, B, "geo", rng.randint(2, 8), 0, rng.randint(n, 8 * n))
        return _solve(S, n, B, "uniform", rng.randint(2, 8), rng.choice([200, 1000, 5000]), rng.randint(n, 4 * n),
                      rng.choice([0.0, 0.1]), rng.choice([0.0, 0.1]))
    S, n, B = rng.randint(3, 24), rng.randint(65, 384), rng.randint(1, 4)
    if rng.random() < 0.5:
        return _located(S, n, B, rng.randint(2, 8), rng.randint(n // 2, 2 * n))
    return _solve(S, n, B, "geo", rng.randint(2, 8), 0, rng.randint(n // 2, 2 * n))


# ---------------------------------------------------------------- inputs


class _Rand:
    def __init__(self, seed):
        self.g = torch.Generator("cuda")
        self.g.manual_seed(int(seed) * 2654435761 % (1 << 62) + 17)

    def ints(self, lo, hi, *shape):
        """Uniform whole numbers in [lo, hi]."""
        return torch.randint(lo, hi + 1, shape, generator=self.g, device="cuda", dtype=torch.int32)

    def below(self, share, *shape):
        return torch.rand(shape, generator=self.g, device="cuda") < share

    def normal(self, *shape):
        return torch.randn(shape, generator=self.g, device="cuda")


def _geo(r, B, S, n, cap_hi):
    """Capacities, compute costs, locations and latencies (ms)."""
    lat = torch.triu(r.ints(5, 300, B, LOCATIONS, LOCATIONS), 1)
    lat = lat + lat.transpose(1, 2) + torch.diag_embed(r.ints(1, 5, B, LOCATIONS))
    loc = r.ints(0, LOCATIONS - 1, B, S, n)
    cost = torch.exp(3.0 + 0.5 * r.normal(B, S, n)).round().clamp(5, 200).to(torch.int32)
    return r.ints(1, cap_hi, B, S, n), cost, loc, lat.contiguous()


def _delays(loc, lat):
    B, S, n = loc.shape
    at = loc[:, :-1, :, None].long() * LOCATIONS + loc[:, 1:, None, :]
    return lat.view(B, -1).gather(1, at.view(B, -1)).view(B, S - 1, n, n)


def _instances(r, c):
    """Tensors of a ``solve`` case."""
    B, S, n = c["batch"], c["stages"], c["nodes"]
    zero = torch.zeros(B, n, dtype=torch.int32, device="cuda")
    if c["recipe"] == "geo":
        cap, cost, loc, lat = _geo(r, B, S, n, c["cap_hi"])
        arc, src, snk = _delays(loc, lat), zero, zero
    elif c["recipe"] == "flow":
        _, _, (clo, chi), (alo, ahi) = FLOW_TESTS[c["setting"]]
        cap = r.ints(clo, chi - 1, B, S, n)
        cost = torch.zeros(B, S, n, dtype=torch.int32, device="cuda")
        arc = r.ints(alo, ahi - 1, B, S - 1, n, n)
        src, snk = r.ints(alo, ahi - 1, B, n), r.ints(alo, ahi - 1, B, n)
    else:
        cap, cost = r.ints(1, c["cap_hi"], B, S, n), r.ints(1, c["cost_hi"], B, S, n)
        arc = r.ints(1, c["cost_hi"], B, S - 1, n, n)
        src, snk = zero, zero
        if c["holes"] > 0:
            arc[r.below(c["holes"], B, S - 1, n, n)] = -1
        if c["dead"] > 0:
            cap[r.below(c["dead"], B, S, n)] = 0
    supply = cap.sum((1, 2)).to(torch.int32) if c["supply"] < 0 else \
        torch.full((B,), c["supply"], dtype=torch.int32, device="cuda")
    return {"node_cap": cap, "node_cost": cost, "arc_cost": arc, "supply": supply, "src_cost": src, "snk_cost": snk}


def _churned(r, base, B):
    """Variants of a base instance: each node gone with a variant's own
    probability in [0.1, 0.3], delays between survivors times [0.9, 1.3]."""
    _, S, n = base["node_cap"].shape
    p = 0.1 + 0.2 * torch.rand(B, 1, 1, generator=r.g, device="cuda")
    alive = torch.rand(B, S, n, generator=r.g, device="cuda") >= p
    arc = base["arc_cost"].expand(B, S - 1, n, n)
    both = alive[:, :-1, :, None] & alive[:, 1:, None, :]
    arc = torch.where(both, (arc * r.ints(90, 130, B, S - 1, n, n) + 50) // 100, arc).to(torch.int32)
    grow = lambda k: base[k].expand((B,) + tuple(base[k].shape[1:])).contiguous()
    return {"node_cap": torch.where(alive, base["node_cap"], 0).to(torch.int32), "node_cost": grow("node_cost"),
            "arc_cost": arc.contiguous(), "supply": grow("supply"), "src_cost": grow("src_cost"),
            "snk_cost": grow("snk_cost")}


def _joining(r, c):
    """A base of 96 relays with one empty position per stage, and one
    candidate per stage: link delays and capacities drawn from the setting,
    compute cost = the node's largest link delay + [50, 100)."""
    S, (clo, chi), (alo, ahi) = NODE_TESTS[c["setting"]]
    n0 = 96 // S
    n = n0 + 1
    cap = torch.zeros(1, S, n, dtype=torch.int32, device="cuda")
    cap[:, :, :n0] = r.ints(clo, chi - 1, 1, S, n0)
    arc = torch.full((1, S - 1, n, n), -1, dtype=torch.int32, device="cuda")
    arc[:, :, :n0, :n0] = r.ints(alo, ahi - 1, 1, S - 1, n0, n0)
    src = torch.zeros(1, n, dtype=torch.int32, device="cuda")
    snk = torch.zeros(1, n, dtype=torch.int32, device="cuda")
    src[:, :n0], snk[:, :n0] = r.ints(alo, ahi - 1, 1, n0), r.ints(alo, ahi - 1, 1, n0)
    into = torch.cat([src[:, None, :n0], arc[:, :, :n0, :n0].amax(2)], 1)
    outof = torch.cat([arc[:, :, :n0, :n0].amax(3), snk[:, None, :n0]], 1)
    cost = torch.zeros(1, S, n, dtype=torch.int32, device="cuda")
    cost[:, :, :n0] = torch.maximum(into, outof) + r.ints(50, 99, 1, S, n0)
    base = {"node_cap": cap, "node_cost": cost, "arc_cost": arc, "src_cost": src, "snk_cost": snk,
            "supply": torch.full((1,), c["supply"], dtype=torch.int32, device="cuda")}
    cand = {"cap": r.ints(clo, chi - 1, S, 1).expand(S, S).contiguous(),
            "in_cost": r.ints(alo, ahi - 1, S, S, n), "out_cost": r.ints(alo, ahi - 1, S, S, n),
            "link_cost": r.ints(alo, ahi - 1, S, S), "src_cost": r.ints(alo, ahi - 1, S),
            "snk_cost": r.ints(alo, ahi - 1, S)}
    most = torch.maximum(cand["in_cost"][:, :, :n0].amax(2), cand["out_cost"][:, :, :n0].amax(2))
    cand["cost"] = (most + r.ints(50, 99, S, S)).contiguous()
    return base, cand, n0


def prepare(case, seed):
    r, c = _Rand(seed), case
    s = {"case": c}
    if c["kind"] == "solve":
        s["in"] = _instances(r, c)
        s["solver"] = Solver(c["stages"], c["nodes"], c["batch"])
    elif c["kind"] == "located":
        B, S, n = c["batch"], c["stages"], c["nodes"]
        cap, cost, loc, lat = _geo(r, B, S, n, c["cap_hi"])
        s["in"] = {"node_cap": cap, "node_cost": cost, "location": loc, "latency": lat,
                   "supply": torch.full((B,), c["supply"], dtype=torch.int32, device="cuda")}
        s["solver"] = Solver(S, n, B)
    elif c["kind"] == "churn":
        one = _instances(r, _solve(c["stages"], c["nodes"], 1, "geo", c["cap_hi"], 0, c["supply"]))
        s["solver"] = Solver(c["stages"], c["nodes"], c["batch"])
        s["solver"].solve(**one)
        flows = s["solver"].flows(0, 1)
        s["start"] = {k: flows[k] for k in ("node_flow", "arc_flow", "src_flow", "snk_flow")}
        s["in"] = _churned(r, one, c["batch"])
    elif c["kind"] == "whatif":
        s["base"], s["cand"], s["slot"] = _joining(r, c)
        S, n = s["base"]["node_cap"].shape[1:]
        s["solver"] = Solver(int(S), int(n), c["count"])
    else:
        S, n = FLOW_TESTS[c["setting"]][:2]
        s["in"] = _instances(r, _flow_test(c["setting"], c["batch"]))
        s["slots"] = int(s["in"]["supply"].max())
        s["seed"] = int(seed)
        s["solver"] = Solver(S, n, c["batch"])
    return s


def run(state):
    c, solver = state["case"], state["solver"]
    if c["kind"] == "solve":
        F, cost, status = solver.solve(**state["in"])
    elif c["kind"] == "located":
        F, cost, status = solver.solve_located(**state["in"])
    elif c["kind"] == "churn":
        F, cost, status = solver.resolve_churn(**state["in"], start=state["start"])
    elif c["kind"] == "whatif":
        batch = solver.whatif_expand(state["base"], state["cand"], state["slot"], c["first"], c["count"])
        F, cost, status = solver.solve(**batch)
        best = solver.whatif_best(F, cost, status, c["first"])
        return {"F": F, "cost": cost, "status": status, "best": best}
    else:
        F, cost, status, details = solver.simulate_heuristic(
            **state["in"], rounds=c["rounds"], objective=c["objective"], seed=state["seed"],
            max_slots=state["slots"], details=True)
        return {"F": F, "cost": cost, "status": status, **details}
    return {"F": F, "cost": cost, "status": status}


# ---------------------------------------------------------------- bookkeeping


def _sizes(c):
    if c["kind"] == "whatif":
        S = NODE_TESTS[c["setting"]][0]
        return c["count"], S, 96 // S + 1
    if c["kind"] == "heuristic":
        S, n = FLOW_TESTS[c["setting"]][:2]
        return c["batch"], S, n
    return c["batch"], c["stages"], c["nodes"]


def work(case):
    """Inputs read once and outputs written once; one addition and one
    comparison per link (any method looks at every link cost once)."""
    B, S, n = _sizes(case)
    node, link, out = 2 * S * n + 2 * n + 1, (S - 1) * n * n, 20
    if case["kind"] == "located":
        read = 4 * B * (3 * S * n + LOCATIONS * LOCATIONS + 1)
    elif case["kind"] == "whatif":  # the base and the candidates, read once
        read = 4 * (node + link + 2 * S * S * (n + 1) + S * S)
    elif case["kind"] == "churn":
        read = 4 * B * (node + link) + 4 * (S * n + link + 2 * n)
    else:
        read = 4 * B * (node + link)
    if case["kind"] == "heuristic":
        out += 4 * link + 20 * S * n + 32
        return {"bytes": read + B * out, "flops": 2 * B * case["rounds"] * link}
    return {"bytes": read + B * out, "flops": 2 * B * link}


def tolerance(case):
    """Whole numbers throughout (the heuristic's temperatures are products
    of the same factors in the same order)."""
    return "exact"


# ---------------------------------------------------------------- plain torch


def _plain(x):
    """(F, cost) of a batch by successive shortest paths, label correction in
    stage order, int64."""
    INF = 1 << 60
    cap, nc = x["node_cap"].long(), x["node_cost"].long()
    arc = torch.where(x["arc_cost"] < 0, INF, x["arc_cost"].long())
    B, S, n = cap.shape
    src, snk, supply = x["src_cost"].long(), x["snk_cost"].long(), x["supply"].long()
    dev, row = cap.device, torch.arange(B, device=cap.device)
    flow, link = torch.zeros_like(cap), torch.zeros_like(arc)
    F = torch.zeros(B, dtype=torch.long, device=dev)
    cost = torch.zeros_like(F)
    SPLIT, SRC = n, n + 1
    while True:
        di, do = torch.full_like(cap, INF), torch.full_like(cap, INF)
        pi, po = torch.full_like(cap, SRC), torch.full_like(cap, SRC)
        di[:, 0] = src

        def better(d, p, k, cand, code):
            take = cand < d[:, k]
            d[:, k] = torch.where(take, cand, d[:, k])
            p[:, k] = torch.where(take, code, p[:, k]) if torch.is_tensor(code) else p[:, k].masked_fill(take, code)

        while True:
            before = di.clone(), do.clone()
            for k in range(S):
                if k:
                    v, a = (do[:, k - 1, :, None] + arc[:, k - 1]).min(1)
                    better(di, pi, k, v, a)
                better(do, po, k, torch.where((flow[:, k] < cap[:, k]) & (di[:, k] < INF), di[:, k] + nc[:, k], INF),
                       SPLIT)
            for k in range(S - 1, -1, -1):
                if k < S - 1:
                    back = torch.where((link[:, k] > 0) & (di[:, k + 1, None, :] < INF),
                                       di[:, k + 1, None, :] - arc[:, k], INF)
                    v, a = back.min(2)
                    better(do, po, k, v, a)
                better(di, pi, k, torch.where((flow[:, k] > 0) & (do[:, k] < INF), do[:, k] - nc[:, k], INF), SPLIT)
            if torch.equal(before[0], di) and torch.equal(before[1], do):
                break
        D, last = (do[:, S - 1] + snk).min(1)
        live = (D < INF) & (F < supply)
        if not bool(live.any()):
            return F, cost
        # walk the predecessors of every live instance together, twice: the
        # bottleneck, then the push
        push = supply - F
        for apply in (False, True):
            k, i = torch.full_like(row, S - 1), last.clone()
            out, on = torch.ones_like(live), live.clone()
            while bool(on.any()):
                b, kk, ii, oo = row[on], k[on], i[on], out[on]
                code = torch.where(oo, po[b, kk, ii], pi[b, kk, ii])
                split, start = code == SPLIT, (code == SRC) & ~oo
                fwd, rev = ~split & ~start & ~oo, ~split & oo
                d = push[b]
                sb, fb, rb = split, fwd, rev
                if apply:
                    sign = torch.where(oo, d, -d)
                    flow[b[sb], kk[sb], ii[sb]] += sign[sb]
                    link[b[fb], kk[fb] - 1, code[fb], ii[fb]] += d[fb]
                    link[b[rb], kk[rb], ii[rb], code[rb]] -= d[rb]
                else:
                    room = torch.full_like(d, INF)
                    room[sb] = torch.where(oo, cap[b, kk, ii] - flow[b, kk, ii], flow[b, kk, ii])[sb]
                    room[rb] = link[b[rb], kk[rb], ii[rb], code[rb]]
                    push[b] = torch.minimum(d, room)
                k[b] = kk + rev.long() - fwd.long()
                i[b] = torch.where(split | start, ii, code)
                out[b] = torch.where(split, ~oo, ~oo & fwd)
                on[b] = ~start
        F = torch.where(live, F + push, F)
        cost = torch.where(live, cost + push * D, cost)
        supply = torch.where(live | (F >= supply), supply, F)  # no path left: done


def _expanded(c, base, cand, slot):
    S, n = base["node_cap"].shape[1:]
    S, n, B = int(S), int(n), c["count"]
    at = np.zeros((B, S), np.int64)  # candidate of each stage
    order, left = np.arange(c["first"], c["first"] + B), [list(range(S)) for _ in range(B)]
    for d in range(S):  # lexicographic numbering of (stage of candidate 0, of 1, ...)
        unit = math.factorial(S - 1 - d)
        pick, order = order // unit, order % unit
        for b in range(B):
            at[b, left[b].pop(pick[b])] = d
    at = torch.from_numpy(at).cuda()
    stage = torch.arange(S, device="cuda").expand(B, S)
    x = {k: v.expand((B,) + tuple(v.shape[1:])).clone() for k, v in base.items()}
    x["node_cap"][:, :, slot] = cand["cap"][at, stage]
    x["node_cost"][:, :, slot] = cand["cost"][at, stage]
    for k in range(S):
        if k:
            x["arc_cost"][:, k - 1, :, slot] = cand["in_cost"][at[:, k], k]
        if k < S - 1:
            x["arc_cost"][:, k, slot, :] = cand["out_cost"][at[:, k], k]
    for k in range(S - 1):
        x["arc_cost"][:, k, slot, slot] = cand["link_cost"][at[:, k], at[:, k + 1]]
    x["src_cost"][:, slot] = cand["src_cost"][at[:, 0]]
    x["snk_cost"][:, slot] = cand["snk_cost"][at[:, S - 1]]
    return x


def exact(case, seed):
    B, S, n = _sizes(case)
    if case["kind"] in ("heuristic", "located") or S * n > 200 or B * S * n * n > 6e7:
        return None  # a simulation in Python, or searches by the thousand: minutes
    r = _Rand(seed)
    if case["kind"] == "solve":
        x = _instances(r, case)
    elif case["kind"] == "churn":
        one = _instances(r, _solve(S, n, 1, "geo", case["cap_hi"], 0, case["supply"]))
        x = _churned(r, one, B)
    else:
        x = _expanded(case, *_joining(r, case))
    F, cost = _plain(x)
    out = {"F": F, "cost": cost, "status": torch.zeros(B, dtype=torch.int32, device="cuda")}
    if case["kind"] == "whatif":
        top = torch.nonzero(F == F.max()).view(-1)
        b = int(top[cost[top] == cost[top].min()][0])
        out["best"] = torch.tensor([case["first"] + b, int(F[b]), int(cost[b])], device="cuda")
    return out
