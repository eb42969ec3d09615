"""GPU parity of the matrix-core workgroup kernel with the CPU oracle, bit for bit, at the sizes where
it can go wrong: edges of the 16-vertex target tiles and of the row widths, every beam-width
instantiation and its neighbours, mapping blocks (8 levels) and windows that never become common,
costs inside and outside the matrix operands' range and cost scales that need the coarse passes."""
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


def graph(seed, k, n, p, nel, directed=False):
    if directed:
        return synth.directed_graph(seed, k, n, n, p, p, 4, nel)
    g = synth.er_graph(seed, k, n, n, p, p, 4)
    if nel:
        g.elabel = np.minimum(synth.uniforms(seed, k, 5, g.m) * nel, nel - 1).astype(np.int32)
    return g


def check(ged, gs, pairs, costs, K, directed=False, complete=False):
    graphs, pairs = GraphSet.from_graphs(gs), np.asarray(pairs, np.int64)
    print(f"  case: sizes {[g.n for g in gs][:12]}, K={K}, costs={costs}, directed={directed}, complete={complete}",
          flush=True)
    db = ged.Database(graphs, directed=directed)
    res = ged.kbest(db, pairs, costs, K, with_cand=True, schedule=ged.SCHED_BLOCK,
                    last_level=ged.LAST_COMPLETE if complete else ged.LAST_SELECT)
    db.close()
    d, m, _, cand = oracle.kbest_pairs(graphs, pairs, costs, K, last_complete=complete, directed=directed,
                                       with_cand=True)
    np.testing.assert_array_equal(res.dist, d)
    np.testing.assert_array_equal(res.maps, m)
    np.testing.assert_array_equal(res.cand, cand)


@pytest.mark.parametrize("K", [1, 16, 17, 32, 33, 64, 65, 128, 129, 256, 257, 512, 513, 1024])
@pytest.mark.parametrize("nel", [0, 2, 4])
def test_beam_widths(ged, K, nel):
    """Both sides of every instantiation's K, unlabelled and with one and two label planes."""
    gs = [graph(201, k, n, 0.2, nel) for k, n in enumerate([20, 33, 9, 70, 25, 64])]
    check(ged, gs, [[0, 1], [2, 3], [4, 5], [5, 4], [3, 2]], UNIT if K % 2 else PAPER, K)


@pytest.mark.parametrize("n2", [0, 1, 15, 16, 17, 31, 32, 33, 127, 128, 129, 255, 256, 257, 495, 511, 512])
def test_target_tiles(ged, n2):
    """Targets at the edges of tiles, words and row widths; sources around the mapping blocks."""
    gs = [graph(202, k, n, 0.15, 0) for k, n in enumerate([7, 8, 9, 24])] + [graph(203, 0, n2, 0.15, 0)]
    for K in (5, 40, 200):
        check(ged, gs, [[k, 4] for k in range(4)], PAPER, K, complete=K == 40)


@pytest.mark.parametrize("n2", [1, 31, 32, 33, 64, 65, 128, 129, 200, 256])
@pytest.mark.parametrize("nel", [0, 3])
def test_directed_halves(ged, n2, nel):
    gs = [graph(204, k, n, 0.1, nel, True) for k, n in enumerate([8, 17])] + [graph(205, 0, n2, 0.06, nel, True)]
    for K in (12, 100, 200):
        check(ged, gs, [[0, 2], [1, 2]], PAPER, K, directed=True, complete=K == 100)


# representable in the matrix operands up to a common factor; a ratio that is not; K-th children far
# outside the bytes (coarse passes) in both; more than 2^22 (counts and int32 instead)
COSTS = [(1, 2, 2, 3, 5, 5), (3, 1, 2, 5, 1, 3), (4, 12, 12, 1, 10, 10), (0, 0, 0, 0, 0, 0), (500, 900, 800, 0, 600, 300),
         (1000, 3000, 2500, 700, 1300, 900), (40, 90, 70, 25, 60, 45), (900_001, 800_003, 700_001, 30_011, 20_021, 35_003)]


@pytest.mark.parametrize("costs", COSTS)
@pytest.mark.parametrize("nel", [0, 3])
def test_costs(ged, costs, nel):
    gs = [graph(206, k, n, p, nel) for k, (n, p) in enumerate([(40, 0.3), (70, 0.1), (45, 0.6), (140, 0.2)])]
    for K in (20, 64, 150):
        check(ged, gs, [[0, 1], [2, 3], [1, 2], [0, 0]], costs, K)
    ds = [graph(207, k, n, 0.1, nel, True) for k, n in enumerate([24, 50])]
    check(ged, ds, [[0, 1], [1, 0]], costs, 50, directed=True)


def test_long_windows(ged):
    """Sources longer than the target (only deletions are left at the end), and beams whose members never
    share an ancestor again: two copies of a component, so equal costs keep both halves alive throughout."""
    n = 150
    a, b = np.arange(0, n - 1), np.arange(1, n)
    path = Graph(n, np.zeros(n, np.int32), a.astype(np.int32), b.astype(np.int32), None)
    none = Graph(n, np.zeros(n, np.int32), np.zeros(0, np.int32), np.zeros(0, np.int32), None)
    er = [graph(208, k, m, 0.2, 0) for k, m in enumerate([200, 30])]
    for K in (16, 64, 256):
        check(ged, [path, none] + er, [[0, 0], [1, 1], [0, 1], [1, 0], [2, 3]], UNIT, K)


@pytest.mark.parametrize("n2", [40, 63, 64, 65, 127, 128, 200, 256, 300])
@pytest.mark.parametrize("K", [1, 12, 32, 64])
def test_common_images(ged, n2, K):
    """Long sources and narrow beams: images common to the whole beam leave the target's positions several
    times, down to none left, with one row a vertex, label planes, directed halves and a completed last level."""
    gs = [graph(209, k, n, 0.1, 0) for k, n in enumerate([130, 200])] + [graph(210, 0, n2, 0.1, 0)]
    check(ged, gs, [[0, 2], [1, 2]], PAPER, K, complete=K == 12)
    check(ged, gs, [[0, 2]], (900_001, 800_003, 700_001, 30_011, 20_021, 35_003), K, complete=K == 64)
    if n2 <= 256:
        gs = [graph(211, 0, 150, 0.1, 3), graph(211, 1, n2, 0.1, 3)]
        check(ged, gs, [[0, 1]], PAPER, K)
        ds = [graph(212, 0, 140, 0.05, 3, True), graph(212, 1, n2, 0.05, 3, True)]
        check(ged, ds, [[0, 1]], PAPER, K, directed=True, complete=K == 32)
