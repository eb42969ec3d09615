"""The tuner's saved lines where the workgroup kernel has two forms: a line measured on another kernel, as files of
earlier versions hold them, and a line for a workgroup size that is no configuration of its own, are passed over
(the bin is timed again, with the same results); the line that takes their place is used."""
import numpy as np
import pytest

import oracle
from paper_2605_00830_amd import synth
from paper_2605_00830_amd.synth import GraphSet

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,K,costs", [(70, 100, synth.UNIT_COSTS), (20, 200, (7, 15, 15, 7, 15, 13))])
def test_lines_of_other_kernels_are_passed_over(tmp_path, n, K, costs):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2605_00830_amd import ged
    graphs = GraphSet.from_graphs([synth.er_graph(601, k, n, n, 0.2, 0.2, 4) for k in range(6)])
    pairs = np.array([[0, 1], [2, 3], [4, 5]], np.int64)
    d, m, _ = oracle.kbest_pairs(graphs, pairs, costs, K)
    db = ged.Database(graphs)

    def tune(path):
        plan = ged.Plan(db, pairs, K, schedule=ged.SCHED_BLOCK)
        dist, maps, _ = plan.outputs()
        timed = plan.tune(costs, dist, maps, cache_path=str(path))
        np.testing.assert_array_equal(dist[:len(pairs)].cpu().numpy(), d)
        np.testing.assert_array_equal(maps[:plan.map_size].cpu().numpy(), m)
        plan.close()
        return timed

    first = tmp_path / "first.txt"
    assert tune(first) == 1 and tune(first) == 0
    key = first.read_text().split()[0]
    kind = "m" if n > 32 else "c"
    old = tmp_path / "old.txt"
    old.write_text(f"{key[:key.rindex('|')]} 0 1 256\n" if key.endswith(kind) else f"{key} 0 1 256\n")
    assert tune(old) == 1 and tune(old) == 0
    xl = tmp_path / "xl.txt"
    xl.write_text(f"{key} 0 1 1024\n")
    assert tune(xl) == 1
    db.close()
