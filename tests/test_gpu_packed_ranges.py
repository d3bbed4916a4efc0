"""The packed pass over its whole range against the oracle: every group width
(4, 8 and 16 lanes), shallow and deep pipelines, and the three value ranges it
tells apart (8-bit flows and small costs; 16-bit flows and costs while labels
stay below 2^25; anything beyond, solved one instance per wave), also mixed in
one batch.  All results are whole numbers: no tolerance."""
import numpy as np
import pytest

import mcf_checks as C
import oracle
from gpu_util import gpu_solve
from paper_2509_21221_amd import mcf
from paper_2509_21221_amd import workloads as W

pytestmark = pytest.mark.gpu


def compare(batch, g, certify=8):
    ref = oracle.solve(batch, flows=False, potentials=False)
    for key in ("status", "F", "cost"):
        np.testing.assert_array_equal(g[key], ref[key], err_msg=key)
    for b in [b for b in range(batch.B) if g["status"][b] == 0][:certify]:
        C.certify(batch, b, int(g["F"][b]), int(g["cost"][b]), g["node_flow"][b], g["arc_flow"][b],
                  g["src_flow"][b], g["snk_flow"][b], g["potential"][b])


def expected(batch):
    """Pass of each valid instance: a shallow one outside the packed bounds
    is reported as the fallback's, a deep one always as the LDS pass's."""
    if batch.S > 8:
        return np.full(batch.B, mcf.GWTF_PASS_LDS)
    big = [np.abs(a).reshape(batch.B, -1).max(1, initial=0) for a in
           (batch.node_cost, batch.arc_cost, batch.src_cost, batch.snk_cost)]
    return np.where((batch.supply > 255) | (np.max(big, 0) > 2047), mcf.GWTF_PASS_GLOBAL, mcf.GWTF_PASS_PACKED)


@pytest.mark.parametrize("n", [1, 4, 5, 8, 9, 16])
@pytest.mark.parametrize("S", [1, 2, 8, 9, 16])
def test_shapes_and_value_ranges(S, n):
    """One batch per shape that mixes the three ranges, with missing links and
    deleted nodes; the ranges' own edges (255 and 256, 2047 and 2048, 65,535
    and 65,536 of flow value, labels about 2^25) in its first instances."""
    wide = ((1 << 25) - (1 << 16)) // (2 * S * n + 3)  # largest cost with labels below the 16-bit form's bound
    part = [W.random_small(12, S, n, seed=51 + i, cap_hi=cap, cost_hi=cost, supply_hi=supply, holes=0.1,
                           zero_cap=0.1)
            for i, (cap, cost, supply) in enumerate([(9, 2047, 255), (60, 2047, 255), (300, 50, 3000),
                                                     (7, min(wide, 60000), 90), (7, wide + 1, 40),
                                                     (200000, 30, 400000)])]
    batch = W.concat(part)
    batch.supply[0], batch.supply[1], batch.supply[2] = 255, 256, 2_000_000_000
    batch.node_cost[3, 0, 0], batch.node_cost[4, 0, 0] = 2047, 2048
    batch.node_cost[36, 0, 0], batch.node_cost[37, 0, 0] = wide - 1, wide
    if n > 1:  # a flow value at the 16-bit bound and one above, over two nodes per stage
        for b, extra in ((60, 0), (61, 1)):
            batch.node_cap[b] = 0
            batch.node_cap[b, :, 0], batch.node_cap[b, :, 1] = 65000, 535 + extra
            batch.supply[b] = 1 << 20
            if S > 1:
                batch.arc_cost[b] = 3
    print(f"packed ranges S={S} n={n}", flush=True)
    g = gpu_solve(batch)
    compare(batch, g)
    for b in (36, 37, 48, 60, 61):
        if g["status"][b] == 0:
            C.certify(batch, b, int(g["F"][b]), int(g["cost"][b]), g["node_flow"][b], g["arc_flow"][b],
                      g["src_flow"][b], g["snk_flow"][b], g["potential"][b])
    ok = g["status"] == 0
    np.testing.assert_array_equal(g["passes"][ok], expected(batch)[ok])


@pytest.mark.parametrize("S,n", [(5, 10), (3, 11), (11, 13), (8, 13), (4, 14), (9, 15)])
def test_rows_of_a_relaxation(S, n):
    """Node counts on both sides of the bounds (10, 13 and 16) at which a
    relaxation takes fewer rows than the group has lanes, in each value range."""
    batch = W.concat([W.random_small(9, S, n, seed=81 + i, cap_hi=9, cost_hi=cost, supply_hi=99, holes=0.2,
                                     zero_cap=0.1) for i, cost in enumerate([2047, 20000, 1 << 20])])
    print(f"packed rows S={S} n={n}", flush=True)
    compare(batch, gpu_solve(batch))


@pytest.mark.parametrize("S,n,B", [(3, 3, 1024), (3, 3, 1025), (3, 3, 16400), (5, 7, 8193), (4, 10, 4097),
                                   (12, 4, 2049), (10, 12, 1030)])
def test_instances_per_wave(S, n, B):
    """Batch sizes at which the instances per wave change, the last wave
    partly empty; some instances in the wider range."""
    batch = W.random_small(B, S, n, seed=61, cap_hi=5, cost_hi=300, supply_hi=2 * n + 4, holes=0.1, zero_cap=0.1)
    batch.supply[::97] = 300
    print(f"packed per wave S={S} n={n} B={B}", flush=True)
    compare(batch, gpu_solve(batch))


@pytest.mark.parametrize("S,n,B", [(9, 4, 1024), (9, 4, 1025), (16, 16, 1026), (12, 9, 2051), (16, 3, 4100)])
def test_deep_instances_beyond_the_wide_form(S, n, B):
    """More than 8 stages with costs beyond the 16-bit form, alone in their
    waves (up to 1,024 instances) and in a launch of their own, where every
    third, none and nearly all of a wave's instances are passed on.  The general
    method alone reports the time of the backward sweeps apart."""
    most = (1 << 27) // (2 * S * n + 3)  # labels up to 2^27
    far = W.random_small(B, S, n, seed=63, cap_hi=5, cost_hi=most, supply_hi=9, holes=0.1, zero_cap=0.1)
    far.node_cost[:, 0, 0] = most
    near = W.random_small(B, S, n, seed=64, cap_hi=5, cost_hi=900, supply_hi=9, holes=0.1, zero_cap=0.1)
    near.supply[1::5] = 300
    third = np.arange(B) % 3 == 0
    third[B // 2:] = np.arange(B - B // 2) % 67 != 5
    third[B // 3:B // 2] = False
    for key in ("node_cap", "node_cost", "arc_cost", "src_cost", "snk_cost", "supply"):
        getattr(near, key)[third] = getattr(far, key)[third]
    near.supply[:] = np.maximum(near.supply, 2)
    print(f"packed deep leftovers S={S} n={n} B={B}", flush=True)
    g = gpu_solve(near, stats=True)
    compare(near, g)
    ok = g["status"] == 0
    assert (g["passes"][ok] == mcf.GWTF_PASS_LDS).all()
    several = ok & (g["stats"][:, 0] > 1)  # a second search sweeps backwards
    np.testing.assert_array_equal((g["stats"][:, 5] > 0)[several], third[several])


@pytest.mark.parametrize("S,n,wide", [(8, 8, False), (5, 7, False), (8, 4, False), (12, 8, False), (8, 8, True)])
def test_reverse_link_counter(S, n, wide):
    """The counter of reverse-link relaxations counts links that carry flow: no
    more than one per stage and round while one unit path is in the flow, and
    the same number whether the instance has a group of its own width or, with
    absent nodes added, 16 lanes (the same searches, round by round)."""
    x = W.random_small(1, S, n, seed=65, cap_hi=3, cost_hi=200, supply_hi=9)
    x.supply[:] = 256 + 40 if wide else 40
    two = x.instance(0)
    two.node_cap[:] = np.minimum(two.node_cap, 1)
    two.supply[:] = 2
    padded = W.random_small(1, S, 9, seed=1)
    padded.node_cap[:] = 0
    padded.arc_cost[:] = W.NO_ARC
    for key in ("node_cap", "node_cost", "src_cost", "snk_cost"):
        getattr(padded, key)[..., :n] = getattr(x, key)
    padded.arc_cost[..., :n, :n] = x.arc_cost
    padded.supply[:] = x.supply
    print(f"packed counters S={S} n={n} wide={wide}", flush=True)
    a, b, c = (gpu_solve(y, stats=True)["stats"][0] for y in (x, padded, two))
    np.testing.assert_array_equal(a[:2], b[:2])
    assert a[0] > 1 and a[3] == b[3] > 0
    assert c[0] == 2 and 0 < c[3] <= (S - 1) * c[1]


@pytest.mark.parametrize("S,n,B", [(8, 13, 40320), (16, 16, 4096)])
def test_workspace_without_fallback_state(S, n, B):
    """A handle of a shape that the packed pass finishes holds the flows,
    potentials and counters of its instances and little else."""
    import torch

    each = 4 * (1 + S * n + (S - 1) * n * n + 2 * S * n + 3) + 8 * mcf.STATS_PER_INSTANCE
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    with mcf.Solver(S, n, B):
        held = before - torch.cuda.mem_get_info()[0]
    print(f"packed workspace S={S} n={n} B={B}: {held} bytes held, {each * B} used", flush=True)
    assert held < 1.2 * each * B


def zigzag(S, n):
    """Two unit chains a and d that the first two paths take; the third must
    enter at b, run back along a, over to c, back along d and out through e:
    about 7 S nodes on one path."""
    a, b, c, d, e = range(5)
    x = W.random_small(1, S, n, seed=1, src_snk=False)
    x.node_cap[:] = 1
    x.node_cost[:] = 1
    x.arc_cost[:] = W.NO_ARC
    x.node_cap[0, 0, [c, e]] = 0
    x.node_cap[0, :, 5:] = 0
    x.node_cap[0, S - 1, [b, c]] = 0
    for k in range(S - 1):
        x.arc_cost[0, k, [a, d], [a, d]] = 1
        x.arc_cost[0, k, [b, c, e], [b, c, e]] = 50
    x.arc_cost[0, S - 2, b, a] = x.arc_cost[0, S - 2, c, d] = 50
    x.arc_cost[0, 0, a, c] = x.arc_cost[0, 0, d, e] = 50
    x.supply[:] = 9
    return x


@pytest.mark.parametrize("S,n,wide", [(8, 5, False), (16, 5, False), (16, 16, False), (16, 8, True)])
def test_paths_longer_than_the_listed_nodes(S, n, wide):
    """A path of more nodes than are listed at a time (64) is walked in
    parts; the batch also holds instances with short paths."""
    x = W.concat([zigzag(S, n), W.random_small(9, S, n, seed=62, cap_hi=4, cost_hi=90, supply_hi=30), zigzag(S, n)])
    if wide:
        x.supply[:] += 300
    print(f"packed zigzag S={S} n={n}", flush=True)
    g = gpu_solve(x)
    assert g["F"][0] == 3 and g["F"][10] == 3
    compare(x, g, certify=11)
