"""The cycle-popping kernel (trees popped round by round in LDS) against the serial oracle, bit for
bit: counts in LDS and in the workspace (above 8192 nodes), the last size it takes, work-group
sizes, rounds that change more nodes than a list holds, deep rounds (two cliques joined by one
edge), root sets, stratified entries, batches, the same for the kernel of the meshes, and the calls
that keep the walker teams."""
import numpy as np
import pytest
import torch

import rwcgen as G
from oracle import wilson as W

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2510_20604_amd")


def _barbell(k):
    a, b = np.triu_indices(k, 1)
    src = np.concatenate([a, a + k, [0]])
    dst = np.concatenate([b, b + k, [k]])
    return G.graphs.EdgeList(2 * k, src.astype(np.int32), dst.astype(np.int32), None)


def _graph(name):
    if name == "barbell":
        return _barbell(40)
    if name == "pairs":      # a heavy edge inside every pair of leaves: over a quarter of the nodes on 2-cycles
        k = 600
        hub = np.zeros(k, np.int32)
        a = (1 + 2 * np.arange(k)).astype(np.int32)
        w = np.concatenate([np.full(k, 1.0), np.full(k, 9.0)]).astype(np.float32)
        return G.graphs.EdgeList(2 * k + 1, np.concatenate([hub, a]), np.concatenate([a, a + 1]), w)
    if name == "star":
        return G.star_graph(700)
    n = int(name[2:])
    return G.erdos_renyi_lcc(n, 8, 5) if name[:2] == "er" else G.barabasi_albert(n, 3, 5)


def _check(s, ref, l):
    np.testing.assert_array_equal(P.as_uint64(s["counts"]), ref["visits"])
    np.testing.assert_array_equal(P.as_uint64(s["counts_sq"]), ref["visits_sq"])
    np.testing.assert_array_equal(P.as_uint64(s["tree_hash"][0]), ref["hash"])
    np.testing.assert_array_equal(s["parents"].cpu().numpy(), ref["parents"][[0, l - 1]])
    assert int(P.as_uint64(s["total_steps"])[0]) == int(ref["steps"].sum())


@pytest.mark.parametrize("name,l,weighted,strata", [
    ("er256", 90, True, 0), ("er257", 90, False, 0), ("er1000", 300, False, 0), ("ba1024", 40, True, 64), ("ba4097", 30, False, 0),
    ("ba8192", 20, True, 0), ("ba8193", 20, False, 32), ("ba16385", 8, False, 0), ("ba30000", 6, True, 0), ("barbell", 40, False, 0),
    ("pairs", 50, True, 0),
    ("star", 30, False, 32)])
def test_cycle_pop_is_bit_exact(name, l, weighted, strata):
    g = _graph(name)
    if weighted and g.w is None:
        g = g.with_weights(G.uniform_weights(g.m, 0.5, 2.0, 9))
    Gd = P.Graph(g.n, g.src, g.dst, g.w)
    o = W.OracleCSR(g.n, g.src, g.dst, g.w)
    ref = W.fastwalk_sample(o, o.pivot, 4001, 0, 2, l, want_parents=True, threads=8, strata=strata)
    s = P.sample_forests(Gd, l, 4001, sample_begin=2, dump=[2, l + 1], strata=strata)
    assert s["walk_kernel"] == ("cycle_pop_strata" if strata else "cycle_pop") and s["lds_graphs"] == 1
    _check(s, ref, l)


def test_cycle_pop_root_sets_and_batches():
    g = G.barabasi_albert(9000, 3, 6)
    Gd = P.Graph(g.n, g.src, g.dst)
    o = W.OracleCSR(g.n, g.src, g.dst)
    S = [7, 4000, 8999]
    ref = W.fastwalk_sample(o, S, 5, 0, 0, 12, want_parents=True, threads=8)
    s = P.sample_forests(Gd, 12, 5, roots=S, dump=[0, 11])
    assert s["walk_kernel"] == "cycle_pop"
    _check(s, ref, 12)
    graphs = [G.erdos_renyi_lcc(200, 6, 1), g, G.barabasi_albert(2000, 4, 2)]
    dev = [P.Graph(x.n, x.src, x.dst) for x in graphs]
    b = P.sample_forests(dev, 10, 17, persistent=True, capture=True)
    assert b["walk_kernel"] == "cycle_pop" and b["lds_graphs"] == 3
    off = 0
    for i, x in enumerate(graphs):
        r = W.fastwalk_sample(W.OracleCSR(x.n, x.src, x.dst), dev[i].pivot, 17, i, 0, 10, threads=8)
        np.testing.assert_array_equal(P.as_uint64(b["counts"])[off:off + x.n], r["visits"])
        np.testing.assert_array_equal(P.as_uint64(b["tree_hash"][i]), r["hash"])
        off += x.n


def _rect(a, b):
    ids = np.arange(a * b).reshape(a, b)
    src = np.concatenate([ids[:, :-1].ravel(), ids[:-1].ravel()])
    dst = np.concatenate([ids[:, 1:].ravel(), ids[1:].ravel()])
    return G.graphs.EdgeList(a * b, src.astype(np.int32), dst.astype(np.int32), None)


def _mesh(name):
    if name == "path":
        return G.path_graph(150)
    if name == "tail":           # hubs, and a path that makes the graph deep
        g, k = G.barabasi_albert(3000, 4, 1), 40
        src = np.concatenate([g.src, [0], np.arange(g.n, g.n + k - 1)])
        dst = np.concatenate([g.dst, [g.n], np.arange(g.n + 1, g.n + k)])
        return G.graphs.EdgeList(g.n + k, src.astype(np.int32), dst.astype(np.int32), None)
    return _rect(*(int(x) for x in name.split("x")))


# the classes' edges (2048, 8000 and 20 500 nodes; above, the tree's words are in the workspace), with
# 9 to 13 bits of round in a word (a sweep over all nodes every 2^bits rounds), the last word of the bitmaps whole and not
@pytest.mark.parametrize("name,l,weighted,strata", [
    ("path", 40, False, 0), ("tail", 30, False, 0), ("3x113", 60, True, 64), ("32x64", 30, False, 0), ("3x683", 6, True, 0),
    ("50x160", 12, True, 0), ("53x151", 8, False, 32), ("100x205", 8, False, 0), ("59x349", 8, True, 32), ("180x182", 6, False, 0),
    ("256x257", 4, True, 0)])
def test_mesh_pop_is_bit_exact(name, l, weighted, strata):
    g = _mesh(name)
    if weighted:
        g = g.with_weights(G.uniform_weights(g.m, 0.5, 2.0, 9))
    Gd = P.Graph(g.n, g.src, g.dst, g.w)
    o = W.OracleCSR(g.n, g.src, g.dst, g.w)
    ref = W.fastwalk_sample(o, o.pivot, 4001, 0, 2, l, want_parents=True, threads=8, strata=strata)
    s = P.sample_forests(Gd, l, 4001, sample_begin=2, dump=[2, l + 1], strata=strata)
    assert s["walk_kernel"] == ("mesh_pop_strata" if strata else "mesh_pop") and s["lds_graphs"] == 1
    _check(s, ref, l)


def test_mesh_pop_root_sets_and_mixed_batches():
    g = _rect(90, 91)
    Gd = P.Graph(g.n, g.src, g.dst)
    S = [5, 4100, 8189]
    ref = W.fastwalk_sample(W.OracleCSR(g.n, g.src, g.dst), S, 5, 0, 0, 12, want_parents=True, threads=8)
    s = P.sample_forests(Gd, 12, 5, roots=S, dump=[0, 11])
    assert s["walk_kernel"] == "mesh_pop"
    _check(s, ref, 12)
    graphs = [_rect(40, 45), G.barabasi_albert(2000, 4, 2), _rect(150, 151), g, _rect(60, 61), G.erdos_renyi_lcc(200, 6, 1)]
    dev = [P.Graph(x.n, x.src, x.dst) for x in graphs]
    for _ in range(2):           # the second call replays the captured launches
        b = P.sample_forests(dev, 10, 17, persistent=True, capture=True)
        assert b["walk_kernel"] == "mesh_pop" and b["lds_graphs"] == 6
        off = 0
        for i, x in enumerate(graphs):
            r = W.fastwalk_sample(W.OracleCSR(x.n, x.src, x.dst), dev[i].pivot, 17, i, 0, 10, threads=8)
            np.testing.assert_array_equal(P.as_uint64(b["counts"])[off:off + x.n], r["visits"])
            np.testing.assert_array_equal(P.as_uint64(b["tree_hash"][i]), r["hash"])
            off += x.n


def test_calls_that_keep_the_walker_teams():
    big = G.barabasi_albert(30001, 2, 3)
    mesh = G.grid_with_deletions(9000, 0.1, 3)   # too many trees for its size (below)
    small = G.erdos_renyi_lcc(300, 8, 1)
    er = G.erdos_renyi_lcc(8400, 8, 2)         # no hubs: counts in the workspace, and too many trees
    assert P.sample_forests(P.Graph(er.n, er.src, er.dst), 1400, 3, want_hash=False)["walk_kernel"] == "wilson_team<true>"
    s = P.sample_forests(P.Graph(mesh.n, mesh.src, mesh.dst), 20000, 3, want_hash=False, want_sq=False)
    assert s["walk_kernel"] == "wilson_team<true>"
    for g, kw in ((big, {}), (mesh, {"lds_state": False}), (small, {"walkers_per_tree": 16}), (small, {"lds_state": False}),
                  (small, {"trees_in_flight": 8}), (small, {"path_ring": True})):
        s = P.sample_forests(P.Graph(g.n, g.src, g.dst), 8, 3, **kw)
        assert s["walk_kernel"].startswith("wilson_team"), kw
    with pytest.raises(P.RWCError) as ei:      # a faulty root set leaves trees without a root: reported, none grown
        P.sample_forests(P.Graph(small.n, small.src, small.dst), 40, 4, roots=[small.n, small.n + 1])
    assert ei.value.status == -2


# rounds that follow the changed nodes only: hubs from 2049 nodes on in calls of many trees, wide weights above
# 4096 nodes and in calls of many trees (er4097 and er4098 have one node less); a heavy edge makes hundreds of rounds of one cycle
@pytest.mark.parametrize("name,l,heavy,strata", [("ba2048", 4000, 1.0, 0), ("ba2049", 4000, 1.0, 4096), ("er4098", 12, 2000.0, 0),
                                                 ("er4097", 12, 2000.0, 0), ("ba8192", 12, 2000.0, 32), ("er1000", 20500, 200.0, 0)])
def test_cycle_pop_with_heavy_edges_is_bit_exact(name, l, heavy, strata):
    g = _graph(name)
    w = np.where(np.random.default_rng(3).random(g.m) < 0.01, heavy, 1.0).astype(np.float32)
    Gd = P.Graph(g.n, g.src, g.dst, w)
    assert Gd.csr.weight_ratio == heavy
    o = W.OracleCSR(g.n, g.src, g.dst, w)
    ref = W.fastwalk_sample(o, o.pivot, 4001, 0, 2, l, want_parents=True, threads=8, strata=strata)
    s = P.sample_forests(Gd, l, 4001, sample_begin=2, dump=[2, l + 1], strata=strata)
    assert s["walk_kernel"] == ("cycle_pop_strata" if strata else "cycle_pop")
    _check(s, ref, l)


def test_many_trees_that_keep_the_walker_teams():
    er = G.erdos_renyi_lcc(7000, 8, 2)     # no hubs, above the teams' LDS limit
    ba = G.barabasi_albert(7000, 3, 2)
    w = np.ones(ba.m, np.float32)
    w[ba.m // 2] = 5000.0                  # one heavy edge, in many trees
    most = 16 * torch.cuda.get_device_properties(0).multi_processor_count
    for g, wt, few, many in ((er, None, most, most + 1), (ba, w, 5714, 5715)):
        Gd = P.Graph(g.n, g.src, g.dst, wt)
        a, b = (P.sample_forests(Gd, l, 3, want_hash=False) for l in (few, many))
        assert a["walk_kernel"] == "cycle_pop" and b["walk_kernel"].startswith("wilson_team")
        one = P.sample_forests(Gd, 1, 3, sample_begin=few, want_hash=False)
        assert torch.equal(a["counts"] + one["counts"], b["counts"])


@pytest.mark.parametrize("name", ["340x409", "340x410", "400x500"])
def test_mesh_pop_on_its_largest_meshes(name):
    """Two work-groups a compute unit up to 139 264 nodes, one up to the last size."""
    test_mesh_pop_is_bit_exact(name, 2, name != "340x410", 0)


@pytest.mark.parametrize("n,roots,kernel", [(2048, 1, "cycle_pop"), (2049, 1, "wilson_team"), (6144, 23, "cycle_pop"),
                                            (6400, 24, "wilson_team"), (6400, 25, "cycle_pop")])
def test_many_trees_with_few_roots(n, roots, kernel):
    """One root that is not the pivot, or a few, in calls of more than 40 million tree nodes."""
    g = G.barabasi_albert(n, 3, 2)
    l = 40000000 // n + 1
    Gd = P.Graph(g.n, g.src, g.dst)
    S = [n - 1 - i for i in range(roots)]
    s = P.sample_forests(Gd, l, 3, roots=S, want_hash=False)
    assert s["walk_kernel"].startswith(kernel)
    a = P.sample_forests(Gd, l - 5, 3, roots=S, want_hash=False)
    assert a["walk_kernel"] == "cycle_pop"
    a = P.sample_forests(Gd, 5, 3, sample_begin=l - 5, roots=S, want_hash=False, accumulate=a)
    assert torch.equal(a["counts"], s["counts"]) and torch.equal(a["counts_sq"], s["counts_sq"])
    if roots == 1:
        one = P.sample_forests(Gd, l, 3, root=S[0], want_hash=False)
        assert one["walk_kernel"].startswith(kernel) and torch.equal(one["counts"], s["counts"])
        assert P.sample_forests(Gd, l, 3, root=Gd.pivot, want_hash=False)["walk_kernel"] == "cycle_pop"
