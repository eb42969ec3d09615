"""The single-pair search with the candidate matrix where every partial edit distance fits the histogram but the
bound with the target's insertions does not: parity with the CPU oracle up to the last bins."""
import numpy as np
import pytest

import oracle
from paper_2605_00830_amd import synth
from paper_2605_00830_amd.synth import GraphSet

pytestmark = pytest.mark.gpu


# 30 vertices of 136 or 135 each: the last level's values reach 4080 of 4096
@pytest.mark.parametrize("costs", [(136, 135, 136, 0, 0, 0), (120, 118, 121, 2, 3, 1)])
@pytest.mark.parametrize("K", [700, 5000])
def test_values_up_to_the_last_bin(costs, K):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2605_00830_amd import ged
    g1, g2 = synth.er_graph(404, 0, 30, 30, 0.2, 0.2, 2), synth.er_graph(404, 1, 60, 60, 0.05, 0.05, 2)
    g2.vlabel = (g2.vlabel + 4).astype(np.int32)
    lab = synth.er_graph(404, 2, 5, 5, 0.9, 0.9, 2)
    lab.elabel = np.arange(lab.m, dtype=np.int32) % 2     # (edge labels in the database: the candidate matrix)
    print(f"  case: 30 x 60, K={K}, costs={costs}", flush=True)
    db = ged.Database(GraphSet.from_graphs([g1, g2, lab]))
    dist, mapping, cand = ged.kbest_wide(db, 0, 1, costs, K)
    db.close()
    d, m, c = oracle.kbest(g1, g2, costs, K, with_cand=True)
    assert (dist, cand) == (d, c)
    np.testing.assert_array_equal(mapping, m)
