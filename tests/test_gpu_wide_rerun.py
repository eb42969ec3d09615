"""One single-pair handle run again and again with other costs: what a run clears goes with its costs' bound, so
every run must find its histograms clean whatever ran before (targets of up to 32 vertices; larger ones within the
histogram, past it, and on the candidate matrix), in both last-level modes."""
import numpy as np
import pytest

import oracle
from paper_2605_00830_amd import synth
from paper_2605_00830_amd.synth import GraphSet

pytestmark = pytest.mark.gpu

SMALL, PAPER, LARGE, FAR, ODD = (1, 1, 1, 0, 0, 0), synth.PAPER_COSTS, (90, 60, 80, 3, 4, 5), (2400, 11, 400, 9, 12, 12), \
    (7, 15, 15, 7, 15, 13)


@pytest.mark.parametrize("n1,n2,K", [(1, 3, 5), (12, 14, 40), (9, 32, 3000), (14, 40, 900), (25, 65, 8001)])
@pytest.mark.parametrize("complete", [False, True])
def test_runs_with_other_costs(n1, n2, K, complete):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2605_00830_amd import ged
    gs = [synth.er_graph(701, 0, n1, n1, 0.3, 0.3, 3), synth.er_graph(701, 1, n2, n2, 0.2, 0.2, 3)]
    db = ged.Database(GraphSet.from_graphs(gs))
    wide = ged.Wide(db, 0, 1, K, last_level=ged.LAST_COMPLETE if complete else ged.LAST_SELECT)
    dist, maps, cand = wide.outputs()
    known = {}
    for costs in (LARGE, SMALL, LARGE, FAR, PAPER, FAR, ODD, SMALL, PAPER):
        if costs not in known:
            known[costs] = oracle.kbest(gs[0], gs[1], costs, K, last_complete=complete, with_cand=True)
        print(f"  case: {n1} x {n2}, K={K}, costs={costs}, complete={complete}", flush=True)
        wide.run(costs, dist, maps, cand)
        d, m, c = known[costs]
        assert (int(dist[0]), int(cand[0])) == (d, c)
        np.testing.assert_array_equal(maps[:n1].cpu().numpy(), m)
    wide.close()
    db.close()
