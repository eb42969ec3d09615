"""GPU parity of the single-pair search for targets of up to 32 vertices with the CPU oracle, at the
sizes where it can go wrong: the edges of the target word, of the mapping's words and of a workgroup's
tiles, one to four label planes, and costs on both sides of the histogram's range."""
import numpy as np
import pytest

import oracle
from paper_2605_00830_amd import synth
from paper_2605_00830_amd.synth import GraphSet

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


def graph(k, n, p, nel):
    g = synth.er_graph(301, k, n, n, p, p, 4)
    if nel:
        g.elabel = np.minimum(synth.uniforms(301, k, 5, g.m) * nel, nel - 1).astype(np.int32)
    return g


def check(ged, g1, g2, costs, K, complete):
    print(f"  case: {g1.n} x {g2.n}, K={K}, costs={costs}, complete={complete}", flush=True)
    db = ged.Database(GraphSet.from_graphs([g1, g2]))
    dist, mapping, cand = ged.kbest_wide(db, 0, 1, costs, K,
                                         last_level=ged.LAST_COMPLETE if complete else ged.LAST_SELECT)
    db.close()
    d, m, c = oracle.kbest(g1, g2, costs, K, last_complete=complete, with_cand=True)
    assert (dist, cand) == (d, c)
    np.testing.assert_array_equal(mapping, m)


@pytest.mark.parametrize("n2", [0, 1, 3, 4, 5, 31, 32, 33])
@pytest.mark.parametrize("K", [1, 255, 256, 257, 3000])
def test_target_word(ged, n2, K):
    for k, n1 in enumerate((0, 1, 4, 5, 12)):
        check(ged, graph(k, n1, 0.3, 0), graph(10 + n2, n2, 0.3, 0), PAPER if k % 2 else UNIT, K, k == 3)


@pytest.mark.parametrize("nel", [0, 2, 4, 5, 9])
def test_planes_and_long_mappings(ged, nel):
    """Sources past 32 vertices: mappings of more than eight words, only deletions left at the end."""
    check(ged, graph(50, 33, 0.2, nel), graph(51, 32, 0.2, nel), UNIT, 600, False)
    check(ged, graph(52, 70, 0.1, nel), graph(53, 9, 0.4, nel), PAPER, 300, True)


@pytest.mark.parametrize("costs", [(0, 0, 0, 0, 0, 0), (30, 40, 40, 7, 9, 9), (300, 400, 400, 70, 90, 90), (3, 1, 2, 5, 1, 3)])
def test_costs(ged, costs):
    check(ged, graph(60, 14, 0.3, 3), graph(61, 17, 0.3, 3), costs, 2000, False)


def test_many_tiles(ged):
    """More parent tiles than workgroups of a level: every workgroup owns several."""
    g1, g2 = graph(70, 12, 0.4, 0), graph(71, 13, 0.4, 0)
    db = ged.Database(GraphSet.from_graphs([g1, g2]))
    K = 600_000
    dist, mapping, cand = ged.kbest_wide(db, 0, 1, UNIT, K)
    db.close()
    d, m, c = oracle.kbest(g1, g2, UNIT, K, with_cand=True)
    assert (dist, cand) == (d, c)
    np.testing.assert_array_equal(mapping, m)
