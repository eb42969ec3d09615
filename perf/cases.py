"""Workloads of the library, as a user's program runs them through the Python binding.

Every case is a dict of plain values.  `call` names the entry points a pass takes:

  plan    a kept ged.Plan and its output tensors, run again on the batch (Plan.run)
  paths   pairs that arrive with the call: a plan made and run for them, and the edit
          operations of the mappings it found (ged.Plan, ged.edit_path)
  wide    a kept ged.Wide: one pair, the whole device, large K (Wide.run)
  serve   a running ged.Server: queries submitted, all results collected

and `graphs` the synth.py family the graphs come from (er: random graphs, molecule: sparse
labelled trees with a few rings, directed: random arcs, mix: the serving mix).  All outputs are
whole numbers: distances, mappings, the children evaluated and edit operations.
"""
import math

import numpy as np
import torch

from paper_2605_00830_amd import ged, synth

UNIT, PAPER = synth.UNIT_COSTS, synth.PAPER_COSTS


def _case(name, call, graphs, pairs, n_lo, n_hi, k, p_lo=0.0, p_hi=0.0, vlabels=5, elabels=0, costs="unit",
          last="select", method="tree", query=False):
    c = dict(call=call, graphs=graphs, pairs=pairs, n_lo=n_lo, n_hi=n_hi, k=k, p_lo=p_lo, p_hi=p_hi,
             vlabels=vlabels, elabels=elabels, costs=costs, last=last, method=method, query=query)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one tiny pair, the smallest call: what a program that compares two graphs at a time waits for
        _case("pair_er_8x9_k16", "plan", "er", 1, 8, 9, 16, 0.3, 0.3, vlabels=4),
        # new pairs of small graphs with each call, and the explicit edit operations of each
        _case("edit_paths_er_300pairs_k64", "paths", "er", 300, 10, 30, 64, 0.1, 0.3),
        # the default benchmark batch: many small unlabelled-edge graphs
        _case("batch_er_n10-30_4096pairs_k64", "plan", "er", 4096, 10, 30, 64, 0.1, 0.3),
        # the same amount of directed graphs
        _case("batch_directed_n10-30_4096pairs_k64", "plan", "directed", 4096, 10, 30, 64, 0.05, 0.15),
        # molecule-shaped graphs in disjoint pairs (a distance table between two sets)
        _case("batch_molecule_n10-70_3000pairs_k64", "plan", "molecule", 3000, 10, 70, 64),
        # one molecule against a database (nearest neighbours), paper costs, a wider beam
        _case("query_molecule_n10-70_1x3000_k128", "plan", "molecule", 3000, 10, 70, 128, costs="paper", query=True),
        # middle-sized graphs: beyond the one-wavefront kernels
        _case("batch_er_n65-250_512pairs_k64", "plan", "er", 512, 65, 250, 64, 0.05, 0.3, vlabels=8),
        # the large-graph batch
        _case("stress_er_n100-500_256pairs_k256", "plan", "er", 256, 100, 500, 256, 0.05, 0.5, vlabels=8),
        # the paper's runtime-versus-K experiment at its largest K
        _case("wide_er_n20_k1200000", "wide", "er", 1, 20, 20, 1200000, 0.4, 0.4, vlabels=4, costs="paper"),
        # the paper's runtime-versus-size experiment (K = 5000)
        _case("wide_er_n500_k5000", "wide", "er", 1, 500, 500, 5000, 0.4, 0.4, vlabels=4, costs="paper"),
        # the assignment-based method on the default benchmark's graphs
        _case("bipartite_er_n10-30_4096pairs_k64", "plan", "er", 4096, 10, 30, 64, 0.1, 0.3, method="bipartite"),
        # queries of the serving mix through the server (1% of them 100 to 500 vertices)
        _case("serve_mix_1500queries_k64", "serve", "mix", 1500, 10, 500, 64),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["small", "small", "directed", "molecule", "query", "medium", "large", "wide_small",
                       "wide_large", "bipartite", "paths", "serve"])
    costs = rng.choice(["unit", "paper"])
    last = rng.choice(["select", "select", "complete"])
    el = rng.choice([0, 0, 3])
    if kind == "small":          # any batch of graphs up to 32 vertices
        lo = rng.randint(1, 20)
        return _case(None, "plan", "er", _log(rng, 1, 6000), lo, rng.randint(lo, 32), rng.randint(1, 64), 0.05, 0.5,
                     elabels=el, costs=costs, last=last)
    if kind == "directed":
        if rng.random() < 0.5:
            return _case(None, "plan", "directed", _log(rng, 1, 4096), 5, rng.randint(8, 32), rng.randint(8, 64), 0.05,
                         0.15, elabels=el, costs=costs, last=last)
        return _case(None, "plan", "directed", _log(rng, 1, 300), 33, rng.randint(50, 256), rng.randint(16, 100), 0.01,
                     0.06, elabels=el, costs=costs, last=last)
    if kind == "molecule":
        return _case(None, "plan", "molecule", _log(rng, 20, 3000), 10, rng.randint(33, 70), rng.randint(8, 64),
                     costs=costs, last=last)
    if kind == "query":
        return _case(None, "plan", "molecule", _log(rng, 20, 3000), 10, rng.randint(33, 70), rng.randint(65, 128),
                     costs=costs, last=last, query=True)
    if kind == "medium":
        lo = rng.randint(33, 100)
        hi = rng.randint(lo, 250)
        return _case(None, "plan", "er", _log(rng, 1, 500), lo, hi, _log(rng, 16, 256 if hi > 128 else 1024), 0.05, 0.3,
                     vlabels=8, elabels=el, costs=costs, last=last)
    if kind == "large":
        lo = rng.randint(100, 300)
        return _case(None, "plan", "er", _log(rng, 1, 256), lo, rng.randint(lo, 500), _log(rng, 16, 256), 0.05, 0.5,
                     vlabels=8, costs=costs, last=last)
    if kind == "wide_small":
        n = rng.randint(10, 40)
        return _case(None, "wide", "er", 1, n, n, _log(rng, 1000, 1200000 if n <= 24 else 300000), 0.4, 0.4, vlabels=4,
                     elabels=el, costs="paper", last=last)
    if kind == "wide_large":
        n = rng.randint(80, 500)
        return _case(None, "wide", "er", 1, n, n, _log(rng, 500, 5000), 0.1, 0.5, vlabels=4, costs="paper", last=last)
    if kind == "bipartite":
        lo = rng.randint(5, 20)
        return _case(None, "plan", "er", _log(rng, 1, 4096), lo, rng.randint(lo, 32), rng.randint(8, 64), 0.1, 0.3,
                     elabels=el, costs=costs, method="bipartite")
    if kind == "paths":
        lo = rng.randint(5, 20)
        return _case(None, "paths", "er", _log(rng, 10, 2000), lo, rng.randint(lo, 64), rng.randint(8, 64), 0.1, 0.3,
                     elabels=el, costs=costs, last=last)
    return _case(None, "serve", "mix", _log(rng, 100, 1500), 10, 500, rng.randint(16, 64))


def _graphs(case, seed, count):
    f, lo, hi = case["graphs"], case["n_lo"], case["n_hi"]
    out = []
    for i in range(count):
        if f == "er":
            g = synth.er_graph(seed, i, lo, hi, case["p_lo"], case["p_hi"], case["vlabels"])
            if case["elabels"]:
                draws = synth.uniforms(seed, i, 5, g.m)
                g.elabel = np.minimum(draws * case["elabels"], case["elabels"] - 1).astype(np.int32)
        elif f == "directed":
            g = synth.directed_graph(seed, i, lo, hi, case["p_lo"], case["p_hi"], case["vlabels"], case["elabels"])
        elif f == "molecule":
            g = synth.molecule_graph(seed, i, lo, hi)
        else:
            g = synth.mix_graph(seed, i)
        out.append(g)
    return synth.GraphSet.from_graphs(out)


def _room(entries):
    """A mapping buffer for batches of any graphs of the case's sizes; what a batch leaves free keeps -2."""
    return torch.full((entries,), -2, dtype=torch.int32, device="cuda")


def prepare(case, seed):
    P, K = case["pairs"], case["k"]
    st = {"case": case, "K": K, "costs": UNIT if case["costs"] == "unit" else PAPER,
          "last": ged.LAST_COMPLETE if case["last"] == "complete" else ged.LAST_SELECT}
    if case["query"]:    # graph 0 against every other
        gs = _graphs(case, seed, P + 1)
        pairs = np.stack([np.zeros(P, np.int64), np.arange(1, P + 1, dtype=np.int64)], 1)
    else:
        gs = _graphs(case, seed, 2 * P)
        pairs = np.stack([np.arange(0, 2 * P, 2, dtype=np.int64), np.arange(1, 2 * P, 2, dtype=np.int64)], 1)
    if case["call"] == "serve":   # the first half is the database, the second the queries
        st["db"] = ged.Database(gs.slice(0, P))
        st["queries"] = gs.slice(P, 2 * P)
        st["targets"] = (np.arange(P, dtype=np.int64) * 7919) % P
        st["recs"], st["keep"] = ged.pack_queries(st["queries"])
        st["offsets"] = np.concatenate([[0], np.cumsum(st["queries"].n, dtype=np.int64)])
        st["dist"], st["map"] = np.empty(P, np.int32), np.full(P * case["n_hi"], -2, np.int32)
        st["server"] = ged.Server(st["db"], K, st["costs"], streams=2)
        return st
    st["db"] = ged.Database(gs, directed=case["graphs"] == "directed")
    st["pairs"] = pairs
    if case["call"] == "plan":
        st["plan"] = ged.Plan(st["db"], pairs, K, last_level=st["last"],
                              method=ged.METHOD_BIPARTITE if case["method"] == "bipartite" else ged.METHOD_TREE)
        dist, _, cand = st["plan"].outputs(with_cand=True)
        st["out"] = dist, _room(P * case["n_hi"]), cand
    elif case["call"] == "wide":
        st["wide"] = ged.Wide(st["db"], 0, 1, K, last_level=st["last"])
        st["out"] = st["wide"].outputs()
    else:
        n = case["n_hi"]
        st["map"] = _room(P * n)
        st["ops"] = np.full((P * (2 * n + math.ceil(case["p_hi"] * n * (n - 1))), 6), -2, np.int32)
    return st


def _serve(st):
    srv, off = st["server"], st["offsets"]
    tickets = srv.submit_batch(st["recs"], st["targets"])
    dist, maps = st["dist"], st["map"]
    left = len(tickets)
    while left:
        got, d, _, m = srv.collect(with_maps=True)
        q = np.searchsorted(tickets, got)
        dist[q] = d
        at = 0
        for k in q:
            n = int(off[k + 1] - off[k])
            maps[off[k]:off[k + 1]] = m[at:at + n]
            at += n
        left -= len(got)
    return {"dist": dist, "map": maps}


def run(st):
    call, costs = st["case"]["call"], st["costs"]
    if call == "plan":
        dist, maps, cand = st["out"]
        st["plan"].run(costs, dist, maps, cand)
        return {"dist": dist, "map": maps, "cand": cand}
    if call == "wide":
        dist, maps, cand = st["out"]
        st["wide"].run(costs, dist, maps, cand)
        return {"dist": dist, "map": maps, "cand": cand}
    if call == "serve":
        return _serve(st)
    plan = ged.Plan(st["db"], st["pairs"], st["K"], last_level=st["last"])
    dist, maps = torch.empty(len(st["pairs"]), dtype=torch.int32, device="cuda"), st["map"]
    plan.run(costs, dist, maps)
    ops, off, cnt = ged.edit_path(st["db"], st["pairs"], costs, maps)
    plan.close()
    used = np.arange(len(ops)) - np.repeat(off[:-1], np.diff(off)) < np.repeat(cnt, np.diff(off))
    ops = ops[used]
    st["ops"][:len(ops)] = ops
    return {"dist": dist, "map": maps, "count": cnt, "ops": st["ops"]}


def _children(n1, n2, K):
    """Children of a search of about these sizes: every parent's free target vertices and its deletion."""
    total, beam = 0, 1
    for i in range(n1):
        free = max(n2 - i, 0) + 1
        total += beam * free
        beam = min(K, beam * free)
    return total


def work(case):
    """bytes: each pair's graphs (label and adjacency bits) read once, the outputs written once.  flops: the integer
    operations of scoring each child once (two ANDs and two bit counts per 32 target vertices, and about 16 more)."""
    if case["graphs"] == "mix":
        kinds = [(0.495, 10, 30), (0.495, 10, 70), (0.01, 100, 500)]
    else:
        kinds = [(1.0, case["n_lo"], case["n_hi"])]
    nbytes = flops = 0.0
    for share, lo, hi in kinds:
        n, P = (lo + hi) / 2, case["pairs"] * share
        w = -(-n // 32) * (2 if case["graphs"] == "directed" else 1)
        planes = 2 if case["elabels"] or case["graphs"] in ("molecule", "mix") else 0
        nbytes += P * (2 * (4 * n + 4 * n * w * (1 + planes)) + 4 * n + 12)
        if case["method"] == "bipartite":    # K assignments, each re-solved over an n by 2n matrix from its parent's
            flops += P * case["k"] * n * 2 * n * 8
        else:
            flops += P * _children(int(n), int(n), case["k"]) * (w * (4 + (2 * (planes + 1) if planes else 0)) + 16)
    return {"bytes": nbytes, "flops": flops}


def exact(case, seed):
    """Every output is a whole number, exact already: there is no 64-bit value to be nearer to."""
    return None
