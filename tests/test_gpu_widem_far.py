"""The single-pair search on the matrix cores where a level's K-th child lies past the histogram's 4096 values:
parity with the CPU oracle over many such levels, in the far histogram's first group of values and in later
ones, and the time of the same search with all costs a hundredth (no child past the histogram)."""
import numpy as np
import pytest

import oracle
from paper_2605_00830_amd import synth
from paper_2605_00830_amd.synth import Graph, GraphSet

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ged():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2605_00830_amd import ged as g
    g.load()
    return g


def er(k, n, p, label):
    """A random graph whose vertex labels are label and label + 1: with labels 4 apart no substitution is free."""
    g = synth.er_graph(402, k, n, n, p, p, 2)
    g.vlabel = (g.vlabel + label).astype(np.int32)
    return g


# (n1, n2, p, costs, K): two substitutions (6000) on most levels; the same with edges, so that values spread; three
# substitutions (8700, the third group of values) on the last levels; rows of 3, 16 and 32 words
CASES = [(60, 60, 0.0, (3000, 0, 0, 0, 0, 0), 5000),
         (60, 70, 0.1, (2048, 3, 5, 1, 8, 4), 3000),
         (9, 40, 0.1, (2900, 0, 7, 0, 1, 1), 30000),
         (25, 65, 0.3, (2400, 11, 400, 9, 12, 12), 8001),
         (14, 300, 0.02, (2900, 0, 0, 5, 1, 2), 3700),
         (6, 600, 0.01, (2900, 1, 3, 0, 2, 2), 3500)]


@pytest.mark.parametrize("n1,n2,p,costs,K,complete", [c + (False,) for c in CASES] + [CASES[1] + (True,)])
def test_many_levels_past_the_histogram(ged, n1, n2, p, costs, K, complete):
    g1, g2 = er(0, n1, p, 0), er(1, n2, p, 4)
    print(f"  case: {n1} x {n2}, p={p}, K={K}, costs={costs}, complete={complete}", flush=True)
    db = ged.Database(GraphSet.from_graphs([g1, g2]))
    dist, mapping, cand = ged.kbest_wide(db, 0, 1, costs, K,
                                         last_level=ged.LAST_COMPLETE if complete else ged.LAST_SELECT)
    db.close()
    d, m, c = oracle.kbest(g1, g2, costs, K, last_complete=complete, with_cand=True)
    assert (dist, cand) == (d, c)
    np.testing.assert_array_equal(mapping, m)


def test_time_does_not_go_with_the_costs(ged):
    """The same search twice, once with all costs 100 times as large: its thresholds lie past the histogram on
    most levels, where each child is scored three times instead of twice.  (Counting every child in every
    workgroup took about 25 times as long as the small costs' run.)"""
    import torch
    n, K = 100, 5000
    none = (np.zeros(0, np.int32), np.zeros(0, np.int32), None)
    gs = [Graph(n, np.zeros(n, np.int32), *none), Graph(n, np.ones(n, np.int32), *none)]
    db = ged.Database(GraphSet.from_graphs(gs))
    wide = ged.Wide(db, 0, 1, K)
    took, outs = [], []
    for costs in ((30, 0, 0, 0, 0, 0), (3000, 0, 0, 0, 0, 0)):
        dist, maps, cand = wide.outputs()
        best = 1e9
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            wide.run(costs, dist, maps, cand)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        took.append(best)
        outs.append((int(dist[0]), maps.cpu().numpy(), int(cand[0])))
    wide.close()
    db.close()
    assert outs[0][0] * 100 == outs[1][0] and outs[0][2] == outs[1][2]
    np.testing.assert_array_equal(outs[0][1], outs[1][1])
    print(f"  {took[0]:.3f} ms, {took[1]:.3f} ms", flush=True)
    assert took[1] < 4 * took[0]
