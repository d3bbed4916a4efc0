"""Which form of a pass solves an instance.  The packed solve, the register
pass, the packed churn re-solve and the heuristic each make a first launch with
tight bounds and pass on what it does not hold; results alone do not show who
solved what.  Here a handle makes the first launch only (an exported switch of
the library that is no part of its ABI), and what it leaves must be exactly the
instances outside its bounds, at each bound and one beyond it; the same calls
made in full agree with the oracle."""
import contextlib
import ctypes

import numpy as np
import pytest

import mcf_checks as C
import oracle
from gpu_util import gpu_solve
from oracle import heuristic as H
from paper_2509_21221_amd import mcf
from paper_2509_21221_amd import workloads as W
from test_gpu_churn import FLOW_KEYS, check, churn
from test_gpu_heuristic import gpu_sim

pytestmark = pytest.mark.gpu
PIPE_WIDE = 6  # the register pass's mark for its unscaled variant


@contextlib.contextmanager
def first_only(monkeypatch):
    """Solvers made meanwhile make first launches only."""
    import torch  # noqa: F401  (the library is to share its HIP runtime)

    lib = mcf.load_library()
    lib.gwtf_internal_first_only.argtypes = [ctypes.c_void_p, ctypes.c_int32]
    lib.gwtf_internal_first_only.restype = None
    init = mcf.Solver.__init__

    def limited(self, *args, **kw):
        init(self, *args, **kw)
        lib.gwtf_internal_first_only(self.handle, 1)

    with monkeypatch.context() as m:
        m.setattr(mcf.Solver, "__init__", limited)
        yield


def same_as_oracle(batch, g):
    ref = oracle.solve(batch, flows=False, potentials=False)
    for key in ("status", "F", "cost"):
        np.testing.assert_array_equal(g[key], ref[key], err_msg=key)
    for b in np.flatnonzero(g["status"] == 0):
        C.certify(batch, b, int(g["F"][b]), int(g["cost"][b]), g["node_flow"][b], g["arc_flow"][b],
                  g["src_flow"][b], g["snk_flow"][b], g["potential"][b])


@pytest.mark.parametrize("S,n", [(1, 4), (4, 4), (8, 8), (8, 13), (9, 4), (12, 10), (16, 16)])
def test_packed_solve(monkeypatch, S, n):
    V = 2 * S * n + 3
    far = ((1 << 25) - (1 << 16) - 1) // V  # the largest cost of the 16-bit form
    x = W.random_small(16, S, n, seed=101, cap_hi=4, cost_hi=60, supply_hi=9)
    x.supply[:] = 7
    first = np.ones(16, bool)       # held by the first launch
    general = np.zeros(16, bool)    # beyond the 16-bit form too
    for b, (cost, supply) in {1: (2047, 7), 2: (2048, 7), 3: (far, 7), 4: (far + 1, 7), 5: (60, 255), 6: (60, 256),
                              7: (60, 1 << 30)}.items():
        x.node_cost[b, S - 1, 0] = cost
        x.supply[b] = supply
        first[b] = cost <= 2047 and supply <= 255
        general[b] = cost > far
    for b, value in ((8, 65535), (9, 65536)):  # the flow value, over two nodes of each stage
        x.node_cap[b] = 0
        x.node_cap[b, :, 0], x.node_cap[b, :, 1] = value - 30000, 30000
        x.supply[b] = 1 << 20
        first[b], general[b] = False, value > 65535
    x.snk_cost[10, n - 1] = 2048
    x.src_cost[11, n - 1] = 2047
    first[10] = False
    if S > 1:
        x.arc_cost[12, S - 2, n - 1, 0] = 2048
        first[12] = False
    x.node_cap[13, 0, 0] = -1       # invalid: the first launch reports it
    print(f"forms packed S={S} n={n}", flush=True)
    with first_only(monkeypatch):
        got = gpu_solve(x, flows=False)
    done = mcf.GWTF_PASS_PACKED if S <= 8 else mcf.GWTF_PASS_LDS
    np.testing.assert_array_equal(got["passes"], np.where(first, done, -1))
    g = gpu_solve(x, stats=True)
    same_as_oracle(x, g)
    # of the forms, only the general method times its backward sweeps apart
    several = (g["status"] == 0) & (g["stats"][:, 0] > 1)
    assert several[[1, 2, 3, 4, 5, 6, 7]].all()
    np.testing.assert_array_equal((g["stats"][:, 5] > 0)[several], general[several])


@pytest.mark.parametrize("S,n", [(1, 17), (8, 33), (16, 64), (32, 64)])
def test_register_solve(monkeypatch, S, n):
    V = 2 * S * n + 3
    edge = ((1 << 24) - 1) // (V + 2)  # the largest cost of the keyed variant
    x = W.random_small(8, S, n, seed=102, cap_hi=3, cost_hi=200, supply_hi=3)
    x.supply[:] = 3
    want = np.full(8, mcf.GWTF_PASS_REGISTER)
    for b, cost in ((1, 1022), (2, 1023), (3, edge), (4, edge + 1)):
        x.node_cost[b, S - 1, n - 1] = cost
        want[b] = mcf.GWTF_PASS_REGISTER if cost <= edge else PIPE_WIDE
    if S > 1:
        x.arc_cost[5, 0, 0, n - 1], x.arc_cost[6, 0, 0, n - 1] = 65534, 65535
        want[5] = mcf.GWTF_PASS_REGISTER if 65534 <= edge else PIPE_WIDE
        want[6] = -1
    x.supply[7] = -1
    print(f"forms register S={S} n={n} edge={edge}", flush=True)
    with first_only(monkeypatch):
        got = gpu_solve(x, flows=False)
    np.testing.assert_array_equal(got["passes"], want)
    g = gpu_solve(x)
    same_as_oracle(x, g)
    np.testing.assert_array_equal(g["passes"], np.where(want == -1, mcf.GWTF_PASS_GLOBAL, mcf.GWTF_PASS_REGISTER))


@pytest.mark.parametrize("S,n", [(1, 4), (3, 3), (8, 8), (8, 16)])
def test_churn(monkeypatch, S, n):
    prev = W.random_small(16, S, n, seed=103, cap_hi=3, cost_hi=60, supply_hi=9)
    var = W.random_small(16, S, n, seed=104, cap_hi=3, cost_hi=60, supply_hi=9, holes=0.1, zero_cap=0.1)
    first = np.ones(16, bool)
    for b, supply in ((1, 255), (2, 256)):
        var.supply[b] = supply
        first[b] = supply <= 255
    for b, cost in ((3, 2047), (4, 2048)):
        var.node_cost[b, S - 1, n - 1] = cost
        first[b] = cost <= 2047
    for b, flow in ((5, 255), (6, 256)):    # the start flow's value
        prev.node_cap[b] = 300
        prev.supply[b] = flow
        first[b] = flow <= 255
    var.snk_cost[7, 0], var.src_cost[8, 0] = 2047, 2048
    first[8] = False
    var.node_cap[9] = 400                   # capacities have no bound
    if S > 1:
        var.arc_cost[10, 0, n - 1, 0] = 2048
        first[10] = False
    var.node_cap[11, 0, 0] = -1             # invalid input is the general form's
    first[11] = False
    start = {k: oracle.solve(prev)[k].copy() for k in FLOW_KEYS}
    start["node_flow"][12, 0, 0] += 1
    start["src_flow"][13, 0] = -1
    first[12] = first[13] = False
    print(f"forms churn S={S} n={n}", flush=True)
    with first_only(monkeypatch):
        status = churn(var, start)[2]
    np.testing.assert_array_equal(status, np.where(first, 0, -1))
    F, cost, status, out, _ = churn(var, start)
    ref = oracle.solve(var)
    bad = np.isin(np.arange(16), (12, 13))
    assert (status[bad] == 1).all() and not F[bad].any() and not cost[bad].any() and not out["node_flow"][bad].any()
    keep = np.flatnonzero(~bad)
    check(var.subset(keep), F[keep], cost[keep], status[keep], {k: v[keep] for k, v in out.items()},
          {k: v[keep] for k, v in ref.items() if k != "threads"}, certify_first=len(keep))


def long_zigzag(S, m, spare, n):
    """m unit chains that carry flow, m + 1 that cannot reach both ends alone:
    one more unit runs forth along each of these and back along each of those,
    about m (3 S - 2) + S nodes.  `spare` (0 or 1) adds a chain that carries a unit
    too; the rest of the n nodes of a stage are absent."""
    x = W.random_small(1, S, n, seed=1, src_snk=False)
    x.node_cap[:] = x.node_cost[:] = 1
    x.arc_cost[:] = W.NO_ARC
    back, forth = range(m), range(m, 2 * m + 1)
    for i in back:
        x.arc_cost[0, :, i, i] = 1
        x.arc_cost[0, S - 2, forth[i], i] = x.arc_cost[0, 0, i, forth[i + 1]] = 50
    for i in forth:
        x.arc_cost[0, :, i, i] = 50
    x.node_cap[0, :, 2 * m + 1 + spare:] = 0
    x.node_cap[0, 0, list(forth[1:])] = x.node_cap[0, S - 1, list(forth[:-1])] = 0
    if spare:
        x.arc_cost[0, :, 2 * m + 1, 2 * m + 1] = 1
    x.supply[:] = m + spare
    return x


@pytest.mark.parametrize("spare", [0, 1])
def test_churn_paths_and_cycles_longer_than_the_list(monkeypatch, spare):
    """A re-solve whose augmenting path (or, when a spare chain becomes dear,
    negative cycle) holds more than the 64 nodes that the packed form lists goes
    to the general form; its neighbours in the wave, short zigzags among them,
    do not."""
    prev = W.concat([long_zigzag(8, m, spare, 12) for m in (5, 1, 5, 2)])
    var = prev.subset(range(4))
    if spare:
        for b, m in enumerate((5, 1, 5, 2)):
            var.arc_cost[b, :, 2 * m + 1, 2 * m + 1] = 2000
    else:
        var.supply = prev.supply + 1
    ref0, ref = oracle.solve(prev), oracle.solve(var)
    assert (ref0["F"] == prev.supply).all() and (ref["F"] == var.supply).all()
    start = {k: ref0[k] for k in FLOW_KEYS}
    print(f"forms churn zigzag spare={spare}", flush=True)
    with first_only(monkeypatch):
        status = churn(var, start)[2]
    np.testing.assert_array_equal(status, [-1, 0, -1, 0])
    F, cost, status, out, work = churn(var, start)
    check(var, F, cost, status, out, ref, certify_first=4)
    assert (work[:, 1 if spare else 2] > 0).all()


@pytest.mark.parametrize("S,n", [(1, 64), (3, 4), (8, 5)])
def test_heuristic(monkeypatch, S, n):
    x = W.random_small(12, S, n, seed=105, cap_hi=3, cost_hi=20, supply_hi=40)
    first = np.ones(12, bool)
    for b, cap in ((1, 32), (2, 33), (3, 200)):
        x.node_cap[b, S - 1, n - 1] = cap
        first[b] = cap <= 32
    x.node_cap[4, 0, 0] = -1    # invalid: the first launch reports it
    x.node_cap[5, 0, 0] = 5000  # more than max_slots
    print(f"forms heuristic S={S} n={n}", flush=True)
    with first_only(monkeypatch):
        got = gpu_sim(x, 20, "sum", 7, 4096)
    np.testing.assert_array_equal(got["status"], np.where(first, [0, 0, 0, 0, 1, 1] + [0] * 6, -1))
    g, r = gpu_sim(x, 20, "sum", 7, 4096), H.simulate(x, rounds=20, objective="sum", seed=7, max_slots=4096)
    for key in ("F", "cost", "status", "node_flow", "arc_flow", "used"):
        np.testing.assert_array_equal(g[key], r[key], err_msg=key)
