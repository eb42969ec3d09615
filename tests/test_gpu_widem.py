"""GPU parity of the single-pair search on the matrix cores (unlabelled edges, targets past 32 vertices)
with the CPU oracle, at the sizes where it can go wrong: the edges of the target's words and row widths,
of the beam's groups and of the mapping blocks, windows that never become common, costs the matrix
operands hold and costs they do not, and a threshold past the histogram's range."""
import numpy as np
import pytest

import oracle
from paper_2605_00830_amd import synth
from paper_2605_00830_amd.synth import Graph, GraphSet

pytestmark = pytest.mark.gpu

UNIT = synth.UNIT_COSTS
PAPER = synth.PAPER_COSTS


@pytest.fixture(scope="module")
def ged():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2605_00830_amd import ged as g
    g.load()
    return g


def graph(k, n, p):
    return synth.er_graph(401, k, n, n, p, p, 4)


def check(ged, g1, g2, costs, K, complete=False):
    print(f"  case: {g1.n} x {g2.n}, K={K}, costs={costs}, complete={complete}", flush=True)
    db = ged.Database(GraphSet.from_graphs([g1, g2]))
    dist, mapping, cand = ged.kbest_wide(db, 0, 1, costs, K,
                                         last_level=ged.LAST_COMPLETE if complete else ged.LAST_SELECT)
    db.close()
    d, m, c = oracle.kbest(g1, g2, costs, K, last_complete=complete, with_cand=True)
    assert (dist, cand) == (d, c)
    np.testing.assert_array_equal(mapping, m)


@pytest.mark.parametrize("n2", [33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 300, 511, 512, 513, 1024])
@pytest.mark.parametrize("K", [1, 63, 64, 65, 700])
def test_target_words(ged, n2, K):
    for k, n1 in enumerate((0, 1, 8, 9, 25)):
        check(ged, graph(k, n1, 0.3), graph(10 + k, n2, 8.0 / n2), PAPER if k % 2 else UNIT, K, k == 3 and n2 < 130)


def test_source_words(ged):
    """Sources at the edges of words and mapping blocks, longer than the target in the last two."""
    for k, (n1, n2) in enumerate([(31, 40), (32, 100), (33, 130), (64, 70), (65, 300), (100, 34), (300, 65)]):
        check(ged, graph(30 + k, n1, 0.2), graph(50 + k, n2, 0.2), PAPER if k % 2 else UNIT, 400, k == 6)


def test_long_windows(ged):
    """Equal costs keep both halves of a symmetric beam alive: blocks that never become common."""
    n = 90
    a, b = np.arange(0, n - 1), np.arange(1, n)
    path = Graph(n, np.zeros(n, np.int32), a.astype(np.int32), b.astype(np.int32), None)
    none = Graph(n, np.zeros(n, np.int32), np.zeros(0, np.int32), np.zeros(0, np.int32), None)
    for g1, g2 in ((path, none), (none, path), (none, none), (path, path)):
        for K in (64, 1000):
            check(ged, g1, g2, UNIT, K)


@pytest.mark.parametrize("costs", [(0, 0, 0, 0, 0, 0), (1, 2, 2, 3, 5, 5), (2, 4, 4, 1, 2, 3), (4, 12, 12, 1, 10, 10),
                                   (3, 1, 2, 5, 1, 7), (40, 90, 70, 20, 60, 40), (300, 400, 400, 70, 90, 90)])
def test_costs(ged, costs):
    check(ged, graph(60, 18, 0.3), graph(61, 45, 0.3), costs, 1500)
    check(ged, graph(62, 18, 0.3), graph(63, 150, 0.1), costs, 300, True)


def test_many_groups(ged):
    """More groups of slots than workgroups of a level: every workgroup owns several."""
    check(ged, graph(70, 7, 0.4), graph(71, 40, 0.3), UNIT, 40_000)


def test_past_the_histogram(ged):
    """All 36004 children of the third level but one survive: the threshold, two deletions, lies past the
    last bin, and the selection counts by itself."""
    check(ged, graph(80, 5, 0.4), graph(81, 33, 0.3), (0, 3000, 0, 0, 0, 0), 36_003)
