"""The single-pair search at the largest beams.  Unlabelled targets past 32 vertices are searched on the matrix
cores or, for the largest K on small targets, with the candidate matrix: parity with the CPU oracle on both sides
of that line; and the matrix-core kernels past 65,536 slots (blocks that no longer join the common mapping) up to
2^21 against the candidate-matrix kernels, which the same pair takes in a database that has edge labels."""
import numpy as np
import pytest

import oracle
from paper_2605_00830_amd import synth
from paper_2605_00830_amd.synth import GraphSet

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ged():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2605_00830_amd import ged as g
    g.load()
    return g


def graph(k, n, p):
    return synth.er_graph(403, k, n, n, p, p, 4)


# 6 x 33 vertices: the line lies at K = 206,569
@pytest.mark.parametrize("K", [206_500, 206_600])
def test_both_sides_of_the_line(ged, K):
    g1, g2 = graph(0, 6, 0.5), graph(1, 33, 0.2)
    print(f"  case: 6 x 33, K={K}", flush=True)
    db = ged.Database(GraphSet.from_graphs([g1, g2]))
    dist, mapping, cand = ged.kbest_wide(db, 0, 1, synth.PAPER_COSTS, K)
    db.close()
    d, m, c = oracle.kbest(g1, g2, synth.PAPER_COSTS, K, with_cand=True)
    assert (dist, cand) == (d, c)
    np.testing.assert_array_equal(mapping, m)


@pytest.mark.parametrize("n1,n2,K", [(20, 36, 70_000), (40, 50, 150_001), (24, 65, 1 << 21), (20, 130, 300_000)])
@pytest.mark.parametrize("complete", [False, True])
def test_beams_past_the_common_mapping(ged, n1, n2, K, complete):
    g1, g2, lab = graph(2, n1, 0.2), graph(3, n2, 0.15), graph(4, 5, 0.9)
    lab.elabel = np.arange(lab.m, dtype=np.int32) % 2
    last = ged.LAST_COMPLETE if complete else ged.LAST_SELECT
    print(f"  case: {n1} x {n2}, K={K}, complete={complete}", flush=True)
    got = []
    for graphs in ([g1, g2], [g1, g2, lab]):
        db = ged.Database(GraphSet.from_graphs(graphs))
        got.append(ged.kbest_wide(db, 0, 1, synth.PAPER_COSTS, K, last_level=last))
        db.close()
    assert got[0][0] == got[1][0] and got[0][2] == got[1][2]
    np.testing.assert_array_equal(got[0][1], got[1][1])
