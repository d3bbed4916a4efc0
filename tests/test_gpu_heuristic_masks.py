"""The heuristic simulation's two kernels at their edges against the oracle,
bit for bit: relays of 31 to 33 slots (slot masks hold 32; instances of both
kinds in one batch), round counts around the eight rounds whose random numbers
are drawn together, and temperatures that decide every move, none, or leave
the range of a float (also the double's: T cools to 0)."""
import numpy as np
import pytest

from oracle import heuristic as H
from paper_2509_21221_amd import workloads as W
from test_gpu_heuristic import KEYS, gpu_sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,n,cap,rounds,t0,alpha", [
    (3, 4, 31, 8, 1.7, 0.95), (3, 4, 32, 9, 1.7, 0.95), (3, 4, 33, 7, 1.7, 0.95), (1, 64, 33, 16, 1.7, 0.95),
    (64, 1, 32, 17, 1.7, 0.95), (8, 5, 3, 1, 1.7, 0.95), (8, 5, 3, 23, 1e-300, 0.95), (8, 5, 3, 40, 9e299, 1.0),
    (8, 5, 3, 200, 50.0, 1e-9), (2, 9, 3, 64, 30.0, 1.05), (2, 32, 6, 24, 8.0, 0.99),
])
def test_mask_and_temperature_edges(S, n, cap, rounds, t0, alpha):
    batch = W.random_small(96, S, n, seed=83 + cap, cap_hi=cap, cost_hi=20, supply_hi=40, holes=0.1, zero_cap=0.1)
    batch.node_cap[::2, 0, 0] = cap
    batch.supply[::3] = batch.node_cap[::3].sum(axis=(1, 2))
    print(f"heuristic masks S={S} n={n} cap={cap} rounds={rounds} T0={t0} alpha={alpha}", flush=True)
    for objective in ("sum", "max"):
        g = gpu_sim(batch, rounds, objective, 7, 4096, t0=t0, alpha=alpha)
        r = H.simulate(batch, rounds=rounds, objective=objective, seed=7, max_slots=4096, T0=t0, alpha=alpha)
        for key in KEYS:
            np.testing.assert_array_equal(g[key], r[key], err_msg=f"{objective} {key}")
