"""The CSR build where its kernels change path: 32- and 64-bit sort keys, rows at the edge of one
group of lanes, one block and the rows taken by whole blocks, tiles of the sort, and breadth-
first levels that are narrow, wide, and expanded from the unreached nodes with short, long and
very long unreached rows.  Checked against the oracle's CSR and SciPy's distances, exactly."""
import numpy as np
import pytest
import scipy.sparse as sp
import scipy.sparse.csgraph as csg

import rwcgen
from oracle import wilson as W

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2510_20604_amd")


def _stars(sizes, links):
    """Stars of the given numbers of leaves; links: (star a, star b, nodes on the path between)."""
    src, dst, centre, nxt = [], [], [], 0
    for s in sizes:
        centre.append(nxt)
        src.append(np.full(s, nxt))
        dst.append(nxt + 1 + np.arange(s))
        nxt += s + 1
    for a, b, k in links:
        path = [centre[a], *range(nxt, nxt + k), centre[b]]
        nxt += k
        src.append(np.array(path[:-1]))
        dst.append(np.array(path[1:]))
    return rwcgen.graphs.EdgeList(nxt, np.concatenate(src).astype(np.int32), np.concatenate(dst).astype(np.int32), None)


def _cases(name):
    rng = np.random.default_rng(11)
    if name == "two_stars":          # the second hub's row (7000, taken by every wave) is unreached on an up level
        return _stars([9000, 7000, 3000, 200], [(0, 1, 2), (0, 2, 3), (0, 3, 4)])
    if name == "rows_255_257":     # the longest row of one group and the shortest of a whole block
        return _stars([255, 256, 257, 15, 16, 17, 1025], [(0, 1, 0), (1, 2, 1), (2, 3, 1), (3, 4, 1), (4, 5, 1), (5, 6, 1)])
    if name == "path_2_16":          # n = 65536: the last size with 32-bit keys
        g = rwcgen.path_graph(65536)
    elif name == "cycle_2_16_1":
        g = rwcgen.cycle_graph(65537)
    elif name == "tile":             # 2m = 2048: one full tile of the sort
        g = rwcgen.cycle_graph(1024)
    elif name == "wide_levels":      # frontiers above the narrow limit on every level
        return rwcgen.grid_with_deletions(300000, 0.02, 5)
    else:
        return rwcgen.rmat_lcc(14, 8, 0.57, 0.19, 0.19, 7)
    perm, flip = rng.permutation(g.m), rng.random(g.m) < 0.5
    a, b = np.where(flip, g.dst, g.src)[perm], np.where(flip, g.src, g.dst)[perm]
    return rwcgen.graphs.EdgeList(g.n, a, b, None)


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("name", ["two_stars", "rows_255_257", "path_2_16", "cycle_2_16_1", "tile", "wide_levels",
                                  "rmat14"])
def test_build_at_the_edges_of_its_kernels(name, weighted):
    g = _cases(name)
    w = rwcgen.uniform_weights(g.m, 0.5, 4.0, 3) if weighted else None
    Gd = P.Graph(g.n, g.src, g.dst, w)
    o = W.OracleCSR(g.n, g.src, g.dst, w)
    nid = Gd.node_id().cpu().numpy()
    perm = np.concatenate([np.arange(o.row_ptr[p], o.row_ptr[p + 1]) for p in nid])
    deg = np.diff(o.row_ptr)[nid]
    want = np.lexsort((np.arange(g.n), -o.strength)) if Gd.internal_order else np.arange(g.n)
    np.testing.assert_array_equal(nid, want)
    np.testing.assert_array_equal(Gd.row_ptr().cpu().numpy(), np.concatenate([[0], np.cumsum(deg)]))
    col = Gd.col().cpu().numpy()
    np.testing.assert_array_equal(nid[col], o.col[perm])
    np.testing.assert_array_equal(Gd.strength().cpu().numpy(), o.strength[nid])
    assert (Gd.pivot, Gd.vol, int(Gd.csr.max_degree)) == (o.pivot, o.vol, int(deg.max()))
    assert np.all(Gd.component().cpu().numpy() == 0)
    rec = Gd.rec().cpu().numpy().reshape(g.n, 16)
    np.testing.assert_array_equal(rec[:, 0], deg)
    np.testing.assert_array_equal(rec[:, 3], col[Gd.row_ptr().cpu().numpy()[:-1]])
    eid = Gd.edge_id().cpu().numpy()
    rows = np.repeat(nid, deg)
    assert np.all(((g.src[eid] == rows) & (g.dst[eid] == nid[col])) | ((g.dst[eid] == rows) & (g.src[eid] == nid[col])))
    if weighted:
        np.testing.assert_array_equal(P.as_uint64(Gd.cdf()), o.cdf[perm])
        np.testing.assert_array_equal(Gd.weight().cpu().numpy(), w[eid])
    order = Gd.bfs_order().cpu().numpy()
    np.testing.assert_array_equal(np.sort(order), np.arange(g.n))
    A = sp.csr_matrix((np.ones(o.col.shape[0]), o.col, o.row_ptr), shape=(g.n, g.n))
    dist = csg.shortest_path(A, unweighted=True, indices=o.pivot)
    assert order[0] == Gd.csr.pivot_index and np.all(np.diff(dist[nid[order]]) >= 0)
    assert Gd.csr.bfs_depth == int(dist.max())
