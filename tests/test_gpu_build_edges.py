"""The CSR build where its kernels change path: 32- and 64-bit sort keys, rows at the edge of one
group of lanes, one block and the rows taken by whole blocks, tiles of the sort, and breadth-
first levels that are narrow, wide, and expanded from the unreached nodes with short, long and
very long unreached rows.  Checked against the oracle's CSR and SciPy's distances, exactly."""
import ctypes

import numpy as np
import pytest
import scipy.sparse as sp
import scipy.sparse.csgraph as csg
import torch

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


def _build_guarded(n, src, dst, w, allow, guard=1 << 22):
    """rwc_build_csr_ex on a workspace with `guard` bytes of a pattern behind it."""
    L = P._lib.lib()
    s, d = (torch.as_tensor(x, dtype=torch.int32).cuda() for x in (src, dst))
    wt = None if w is None else torch.as_tensor(w).cuda()
    size = ctypes.c_size_t()
    assert L.rwc_build_csr_workspace(n, len(src), int(w is not None), ctypes.byref(size)) == 0
    ws = torch.full((size.value + guard,), 0xA5, dtype=torch.uint8, device="cuda")
    csr = P._lib.RwcCsr()
    rc = L.rwc_build_csr_ex(n, len(src), s.data_ptr(), d.data_ptr(), None if wt is None else wt.data_ptr(), allow,
                            ws.data_ptr(), size.value, ctypes.byref(csr), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert bool((ws[size.value:] == 0xA5).all()), "written past the workspace"

    def view(addr, count):
        off = addr - ws.data_ptr()
        return ws[off:off + 4 * count].view(torch.int32).cpu().numpy()
    return rc, csr, view


@pytest.mark.parametrize("n,m,weighted", [(20000, 10, False), (100000, 300, True), (1000000, 100000, False), (65, 1, True)])
def test_build_with_far_more_nodes_than_entries(n, m, weighted):
    """Most nodes isolated: every array by node has to hold n entries where those by entry hold fewer.
    Refused without the flag, and nothing behind the workspace is touched either way."""
    rng = np.random.default_rng(n + m)
    pairs = np.unique(np.sort(rng.integers(0, n, (2 * m, 2)), axis=1), axis=0)
    pairs = rng.permutation(pairs[pairs[:, 0] != pairs[:, 1]])[:m]
    src, dst = pairs[:, 0], pairs[:, 1]
    w = rwcgen.uniform_weights(len(src), 0.5, 4.0, 3) if weighted else None
    assert _build_guarded(n, src, dst, w, 0)[0] == -6
    rc, csr, view = _build_guarded(n, src, dst, w, P._lib.RWC_BUILD_ALLOW_DISCONNECTED)
    assert rc == 0
    A = sp.csr_matrix((np.ones(len(src)), (src, dst)), shape=(n, n))
    count, label = csg.connected_components(A, directed=False)
    smallest = np.full(count, n)
    np.minimum.at(smallest, label, np.arange(n))
    assert csr.components == count
    np.testing.assert_array_equal(view(csr.component, n), smallest[label])
    order, node_id = view(csr.bfs_order, n), view(csr.node_id, n)
    np.testing.assert_array_equal(np.sort(order), np.arange(n))
    dist = csg.shortest_path(A, directed=False, unweighted=True, indices=csr.pivot)
    reached = int(np.isfinite(dist).sum())
    got = dist[node_id[order]]
    assert order[0] == csr.pivot_index and np.all(np.diff(got[:reached]) >= 0)
    assert csr.bfs_depth == int(got[reached - 1])
    assert np.all(np.isinf(got[reached:])) and np.all(np.diff(order[reached:]) > 0)


def test_largest_entry_count():
    """2^30 - 1 edges, the most a graph may have: every node joined to the 1023 that follow it on a ring and
    (almost every one) to the 1024th, and 64 leaves, whose short rows end at entry 2^31 - 2.  Loops over
    the last rows step past 2^31.  The build, and the pivot solve's residual from the ring's sums."""
    N, D, leaves = 1 << 20, 1023, 64
    n, m = N + leaves, (1 << 30) - 1
    node = torch.arange(N, dtype=torch.int32, device="cuda")
    extra = m - N * D - leaves                       # of the 1024th neighbours
    at = torch.arange(leaves, dtype=torch.int32, device="cuda") * 16381 + 5
    src = torch.cat([node.repeat(D), node[:extra], at])
    dst = torch.cat([((node[None, :] + torch.arange(1, D + 1, dtype=torch.int32, device="cuda")[:, None]) % N).flatten(),
                     (node[:extra] + D + 1) % N, node[:leaves] + N])
    assert src.numel() == dst.numel() == m
    Gd = P.Graph(n, src, dst)
    del src, dst
    deg = torch.full((n,), 2 * D, dtype=torch.int64, device="cuda")
    deg[:extra] += 1
    deg[(node[:extra].long() + D + 1) % N] += 1
    deg[at.long()] += 1
    deg[N:] = 1
    assert (Gd.nnz, Gd.internal_order, Gd.components) == (2 * m, 0, 1)
    assert torch.equal(Gd.strength(), deg.double()) and Gd.pivot == int((deg == deg.max()).nonzero()[0])
    ptr = Gd.row_ptr().long()
    assert torch.equal(ptr[1:] - ptr[:-1], deg) and int(ptr[-1]) == 2 * m
    # the longest way: half the ring (2^19) in steps of 1024, and a leaf
    assert 512 <= Gd.csr.bfs_depth <= 514
    assert torch.equal(Gd.bfs_order().sort().values, torch.arange(n, dtype=torch.int32, device="cuda"))
    assert torch.equal(Gd.col()[-leaves:], at)
    e = P.estimate(Gd, torch.ones(n, dtype=torch.int64, device="cuda"), 1)
    h = e["hit"]
    ring = h[:N]
    y = torch.zeros(n, dtype=torch.float64, device="cuda")
    for j in range(1, D + 1):
        y[:N] += ring.roll(j) + ring.roll(-j)
    far = (node[:extra].long() + D + 1) % N
    y[:extra] += ring[far]
    y[far] += ring[:extra]
    y[at.long()] += h[N:]
    y[N:] = ring[at.long()]
    r = deg * h - y - deg
    r[Gd.pivot] = 0.0
    # the solve's 1e-12; rounding of sums of deg terms as large as h; and the drift of a residual updated
    # once an iteration, by as much as a product with a matrix of norm 2 max(deg) rounds
    bound = 1e-12 * float(deg.double().norm()) + 2.0 ** -52 * float((deg * h).norm()) * (64 + 4 * e["iters"])
    assert float(r.norm()) <= bound


@pytest.mark.parametrize("leaves,at", [(15, 14), (17, 16), (200, 199), (256, 255), (257, 0), (2000, 1777)])
def test_weight_ratio(leaves, at):
    """The largest over the smallest weight, wherever in a row they are: among the first sixteen entries, past
    them, and in rows taken by a whole block."""
    w = np.full(leaves, 2.0, np.float32)
    w[at], w[leaves // 2] = 60000.0, 0.75
    g = rwcgen.star_graph(leaves + 1)
    assert P.Graph(g.n, g.src, g.dst, w).csr.weight_ratio == 80000.0
    assert P.Graph(g.n, g.src, g.dst).csr.weight_ratio == 1.0
