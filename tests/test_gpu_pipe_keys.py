"""The stage-pipelined register pass at the edges of its keyed variant,
against the oracle: link costs at the two-rows-per-instruction bound (1022 and
1023), labels at the keyed bound ((V + 2) * max cost = 2^24, one instance below
and one at it), flow lists longer than the entries kept in registers, ragged
shapes with idle waves, and labels that spread more than 1023 over a stage.  All
results are whole numbers: no tolerance."""
import numpy as np
import pytest

import mcf_checks as C
import oracle
from gpu_util import gpu_solve
from paper_2509_21221_amd import workloads as W

pytestmark = pytest.mark.gpu


def compare(batch, g):
    ref = oracle.solve(batch, flows=False, potentials=False)
    for key in ("status", "F", "cost"):
        np.testing.assert_array_equal(g[key], ref[key], err_msg=key)
    for b in range(batch.B):
        if g["status"][b] == 0:
            C.certify(batch, b, int(g["F"][b]), int(g["cost"][b]), g["node_flow"][b], g["arc_flow"][b],
                      g["src_flow"][b], g["snk_flow"][b], g["potential"][b])


@pytest.mark.parametrize("S,n", [(1, 17), (3, 64), (8, 33), (9, 17), (16, 64), (17, 31), (31, 20), (32, 64)])
@pytest.mark.parametrize("holes", [0.0, 0.15])
def test_cost_and_label_edges(S, n, holes):
    edge = ((1 << 24) - 1) // (2 * S * n + 3 + 2)  # the largest cost the keys hold
    part = []
    for i, cost in enumerate((1022, 1023, 5, min(edge, 65000), min(edge + 1, 65000))):
        x = W.random_small(2, S, n, seed=71 + i, cap_hi=9, cost_hi=cost, supply_hi=6 * n, holes=holes, zero_cap=0.05)
        x.node_cost[:, 0, 0] = cost
        if S > 1:
            x.arc_cost[:, 0, 0, :] = cost
        part.append(x)
    batch = W.concat(part)
    batch.supply[:] = 5 * n
    print(f"pipe keys S={S} n={n} holes={holes}", flush=True)
    compare(batch, gpu_solve(batch))


@pytest.mark.parametrize("S,n", [(6, 40), (14, 20), (32, 48)])
def test_long_lists_and_spread_labels(S, n):
    """Small costs and large capacities give exits many partners; a stage
    whose nodes' costs differ by up to 1022 spreads the labels beyond what 16
    bits of key tell apart."""
    x = W.random_small(6, S, n, seed=77, cap_hi=40, cost_hi=3, supply_hi=900)
    x.supply[:] = 12 * n
    x.node_cost[3:, ::2] = np.random.default_rng(5).integers(0, 1023, x.node_cost[3:, ::2].shape)
    x.src_cost[3:] = np.random.default_rng(6).integers(0, 1023, x.src_cost[3:].shape)
    print(f"pipe lists S={S} n={n}", flush=True)
    compare(x, gpu_solve(x))
