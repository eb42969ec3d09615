"""GPU parity of the matrix-core workgroup kernel with the CPU oracle where a level's children lie more than
2^30 apart: the least child's reduction must not wrap (survivors past the beam would be written)."""
import numpy as np
import pytest

import oracle
from paper_2605_00830_amd.synth import Graph, GraphSet

pytestmark = pytest.mark.gpu


def plain(n, src=(), dst=()):
    return Graph(n, np.zeros(n, np.int32), np.asarray(src, np.int32), np.asarray(dst, np.int32), None)


# One target edge that costs 1.5e9 to insert.  The beam fills before 2 i + 1 partial mappings without both of
# its ends exist, so T sits past 1.5e9 above the least parent until they do; at that level the K-th child falls
# back below the range that the previous T suggests.  (K, n1): levels 31 and 127 of 64- and 256-slot beams.
@pytest.mark.parametrize("K,n1", [(64, 100), (256, 200)])
@pytest.mark.parametrize("n2", [2, 40])
def test_children_far_apart(K, n1, n2):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2605_00830_amd import ged
    gs = GraphSet.from_graphs([plain(n1), plain(n2, [0], [1])])
    costs = (0, 1, 0, 0, 0, 1_500_000_000)
    db = ged.Database(gs)
    res = ged.kbest(db, np.array([[0, 1]]), costs, K, with_cand=True, schedule=ged.SCHED_BLOCK)
    db.close()
    d, m, _, cand = oracle.kbest_pairs(gs, np.array([[0, 1]]), costs, K, with_cand=True)
    np.testing.assert_array_equal(res.dist, d)
    np.testing.assert_array_equal(res.maps, m)
    np.testing.assert_array_equal(res.cand, cand)
