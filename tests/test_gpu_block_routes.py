"""GPU parity with the CPU oracle on both sides of the lines between the workgroup kernel's two forms (matrix cores,
candidate matrix): beam widths, small targets, long sources, directed and labelled graphs, few and many pairs, costs
inside and outside the matrix operands; the same through a captured graph, the allocation-free call and the server."""
import numpy as np
import pytest

import oracle
from paper_2605_00830_amd import synth
from paper_2605_00830_amd.synth import GraphSet

pytestmark = pytest.mark.gpu

FAST, COUNTS = synth.PAPER_COSTS, (7, 15, 15, 7, 15, 13)


@pytest.fixture(scope="module")
def ged():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2605_00830_amd import ged as g
    g.load()
    return g


def graph(k, n, p, nel, directed):
    if directed:
        return synth.directed_graph(501, k, n, n, p, p, 4, nel)
    g = synth.er_graph(501, k, n, n, p, p, 4)
    if nel:
        g.elabel = np.minimum(synth.uniforms(501, k, 5, g.m) * nel, nel - 1).astype(np.int32)
    return g


def want(graphs, pairs, costs, K, directed):
    d, m, _, cand = oracle.kbest_pairs(graphs, pairs, costs, K, directed=directed, with_cand=True)
    return d, m, cand


def check(ged, gs, pairs, costs, K, directed=False):
    graphs, pairs = GraphSet.from_graphs(gs), np.asarray(pairs, np.int64)
    print(f"  case: {len(pairs)} pairs, sizes {[g.n for g in gs][:8]}, K={K}, costs={costs}, directed={directed}", flush=True)
    db = ged.Database(graphs, directed=directed)
    res = ged.kbest(db, pairs, costs, K, with_cand=True, schedule=ged.SCHED_BLOCK)
    db.close()
    d, m, cand = want(graphs, pairs, costs, K, directed)
    np.testing.assert_array_equal(res.dist, d)
    np.testing.assert_array_equal(res.maps, m)
    np.testing.assert_array_equal(res.cand, cand)


@pytest.mark.parametrize("K", [64, 65, 128, 129, 256, 257, 512, 513, 640, 641, 896, 897])
@pytest.mark.parametrize("nel", [0, 3])
@pytest.mark.parametrize("directed", [False, True])
def test_few_pairs(ged, K, nel, directed):
    gs = [graph(k, n, 0.2, nel, directed) for k, n in enumerate([12, 32, 9, 33, 14, 64, 10, 70])]
    for costs in (FAST, COUNTS):
        check(ged, gs, [[0, 1], [2, 3], [4, 5], [6, 7], [4, 2]], costs, K, directed)


@pytest.mark.parametrize("K", [16, 17, 32, 33, 65, 256, 257, 513, 897])
@pytest.mark.parametrize("nel,directed", [(0, False), (3, False), (0, True), (3, True)])
def test_many_pairs(ged, K, nel, directed):
    """520 pairs: 256-thread workgroups, more pairs than a persistent grid holds."""
    gs = [graph(k, 2 + k % 6, 0.4, nel, directed) for k in range(40)]
    pairs = [[(7 * k) % 40, (3 * k + 11) % 40] for k in range(520)]
    for costs in (FAST, COUNTS):
        check(ged, gs, pairs, costs, K, directed)


@pytest.mark.parametrize("n1", [128, 129, 200, 201, 300, 301])
def test_long_sources(ged, n1):
    """257 pairs of one long source: more pairs than CUs."""
    gs = [graph(0, n1, 0.03, 0, False)] + [graph(k, 1 + k % 2 * 40, 0.1, 0, False) for k in (1, 2)]
    check(ged, gs, [[0, 1 + k % 2] for k in range(2)], COUNTS, 128)
    gs = [graph(0, n1, 0.03, 0, False)] + [graph(k, 2 + k % 3, 0.5, 0, False) for k in range(1, 4)]
    check(ged, gs, [[0, 1 + k % 3] for k in range(257)], COUNTS, 65)


def test_capture_noalloc_and_server(ged):
    import torch
    gs = [graph(k, n, 0.2, 0, False) for k, n in enumerate([20, 30, 9, 25, 40, 60])]
    graphs, K = GraphSet.from_graphs(gs), 300
    pairs = np.array([[0, 1], [2, 3], [4, 5], [1, 0], [5, 2]], np.int64)
    db = ged.Database(graphs)
    for costs in (FAST, COUNTS):
        d, m, cand = want(graphs, pairs, costs, K, False)
        plan = ged.Plan(db, pairs, K)
        dist, maps, cnt = plan.outputs(with_cand=True)
        other = torch.empty_like(dist), torch.empty_like(maps)
        s = torch.cuda.Stream()
        plan.capture(costs, dist, maps, cnt, stream=s)
        for _ in range(3):
            with torch.cuda.stream(s):
                dist.fill_(-7)
                maps.fill_(-7)
                cnt.fill_(-7)
            plan.replay(stream=s)
            s.synchronize()
            np.testing.assert_array_equal(dist[:len(pairs)].cpu().numpy(), d)
            np.testing.assert_array_equal(maps[:plan.map_size].cpu().numpy(), m)
            np.testing.assert_array_equal(cnt[:len(pairs)].cpu().numpy(), cand)
            plan.run(FAST if costs is COUNTS else COUNTS, *other)   # the other form, on the same workspace
            torch.cuda.synchronize()
        ged.kbest_noalloc(db, pairs, costs, K, dist, maps)
        np.testing.assert_array_equal(dist[:len(pairs)].cpu().numpy(), d)
        np.testing.assert_array_equal(maps[:plan.map_size].cpu().numpy(), m)
        plan.close()
        server = ged.Server(db, K, costs)
        off = 0
        for k, (a, b) in enumerate(pairs):
            r = server.wait(server.submit(gs[a], int(b)))
            assert int(r[0]) == d[k]
            np.testing.assert_array_equal(np.asarray(r[1]), m[off:off + gs[a].n])
            off += gs[a].n
        server.close()
    db.close()
