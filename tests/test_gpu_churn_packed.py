"""The packed churn re-solve (S <= 8, n <= 16) at the edges of what it holds,
against the oracle's cold solve: every group width, and batches that mix
instances it solves with ones it passes on to the general form (supply or flow
above 255, a cost above 2047) and ones whose start flow is invalid."""
import numpy as np
import pytest

import oracle
from paper_2509_21221_amd import workloads as W
from test_gpu_churn import FLOW_KEYS, check, churn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 4, 5, 8, 9, 16])
@pytest.mark.parametrize("S", [1, 2, 8])
def test_value_ranges_in_one_batch(S, n):
    kinds = [(4, 60, 40), (9, 2047, 255), (300, 2047, 255), (300, 40, 900), (5, 9000, 60)]
    prev = W.concat([W.random_small(16, S, n, seed=91 + i, cap_hi=c, cost_hi=w, supply_hi=s)
                     for i, (c, w, s) in enumerate(kinds)])
    var = W.concat([W.random_small(16, S, n, seed=191 + i, cap_hi=c, cost_hi=w, supply_hi=s, holes=0.15, zero_cap=0.15)
                    for i, (c, w, s) in enumerate(kinds)])
    var.supply[0], var.supply[1], var.supply[2] = 255, 256, 0
    var.node_cost[3, 0, 0], var.node_cost[4, 0, 0] = 2047, 2048
    var.node_cap[5] = 0            # everything deleted: the whole start flow is stripped
    var.node_cap[6, 0, 0] = -1     # invalid input
    start = {k: oracle.solve(prev)[k].copy() for k in FLOW_KEYS}
    start["node_flow"][7, 0, 0] += 1   # not conserved
    start["src_flow"][8, 0] = -1       # negative
    print(f"churn packed S={S} n={n}", flush=True)
    F, cost, status, out, work = churn(var, start)
    ref = oracle.solve(var)
    for b in (7, 8):
        assert status[b] == 1 and F[b] == 0 and cost[b] == 0 and not out["node_flow"][b].any()
    keep = [b for b in range(var.B) if b not in (7, 8)]
    pick = lambda d: {k: v[keep] for k, v in d.items()}
    check(var.subset(keep), F[keep], cost[keep], status[keep], pick(out), pick({k: ref[k] for k in ref if k != "threads"}),
          certify_first=len(keep))
    assert F[5] == 0
    assert (work[5, 0] > 0) == bool(start["src_flow"][5].any())


@pytest.mark.parametrize("S,n,B", [(6, 8, 1025), (6, 3, 16385), (7, 12, 2049), (8, 8, 1)])
def test_shared_start_and_batch_sizes(S, n, B):
    """One start flow for the whole batch, at batch sizes where the instances
    per wave change and the last wave is partly empty."""
    base = W.random_small(1, S, n, seed=95, cap_hi=5, cost_hi=200, supply_hi=3 * n)
    base.supply[:] = 3 * n
    var = W.random_small(B, S, n, seed=96, cap_hi=5, cost_hi=200, supply_hi=3 * n, holes=0.05, zero_cap=0.1)
    var.arc_cost[::2] = base.arc_cost
    b0 = oracle.solve(base)
    print(f"churn packed S={S} n={n} B={B}", flush=True)
    F, cost, status, out, _ = churn(var, {k: b0[k][:1] for k in FLOW_KEYS})
    check(var, F, cost, status, out, oracle.solve(var), certify_first=24)
