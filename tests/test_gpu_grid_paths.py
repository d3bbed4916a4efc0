"""The grid pass's path batches: many exits of the last stage tie, so that one
search gives more paths than a batch takes, paths that no longer fit behind the
others (140 and 400 arcs of 1,024), supplies that end inside a batch, tied
paths that an earlier one blocks, and reverse arcs between them."""
import numpy as np
import pytest

import mcf_checks as C
import oracle
from gpu_util import gpu_solve
from paper_2509_21221_amd import mcf
from paper_2509_21221_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,n,supply,cost_hi", [(2, 65, 200, 0), (2, 130, 17, 0), (3, 129, 16, 1), (70, 66, 90, 0),
                                                (70, 66, 300, 1), (200, 65, 40, 0), (5, 512, 600, 1), (1, 80, 50, 0)])
def test_tied_paths(S, n, supply, cost_hi):
    batch = W.random_small(2, S, n, seed=S + n, cap_hi=3, cost_hi=max(cost_hi, 1), supply_hi=supply, zero_cap=0.1)
    if cost_hi == 0:  # every path costs the same
        for a in (batch.node_cost, batch.arc_cost, batch.src_cost, batch.snk_cost):
            a[:] = 1
    batch.supply[:] = supply
    batch.node_cap[1] = np.minimum(batch.node_cap[1], 1)
    print(f"grid paths S={S} n={n} supply={supply}", flush=True)
    g = gpu_solve(batch)
    ref = oracle.solve(batch, flows=False, potentials=False)
    for key in ("status", "F", "cost"):
        np.testing.assert_array_equal(g[key], ref[key], err_msg=key)
    assert (g["passes"] == mcf.GWTF_PASS_GRID).all()
    for b in range(batch.B):
        C.certify(batch, b, int(g["F"][b]), int(g["cost"][b]), g["node_flow"][b], g["arc_flow"][b],
                  g["src_flow"][b], g["snk_flow"][b], g["potential"][b])
