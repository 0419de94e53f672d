"""The pivot solve in its three forms (one work-group, two launches per iteration with (z, p) pairs,
three launches) at the sizes where they change, with short rows, rows taken by a wave and rows
taken by a block, one grounded node and grounded sets.  Hitting times against SciPy's Jacobi-CG
of the grounded system run to a relative residual of 1e-14, at the 1e-9 that the estimate is held
to elsewhere (the solve stops at 1e-12); the host-checked and the stream-ordered solve agree bit
for bit, and too few iterations are reported by both."""
import numpy as np
import pytest
import scipy.sparse as sp
import scipy.sparse.linalg as spl
import torch

import rwcgen as G

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2510_20604_amd")


def _case(name):
    if name == "k2":
        return G.path_graph(2)
    if name == "star4096":        # one row of 4095 entries, in one work-group
        return G.star_graph(4096)
    if name == "er4096":          # the largest n of one work-group; unit weights only fit (weights: the pairs)
        return G.erdos_renyi_lcc(4096, 6, 3)
    if name == "er4200":
        return G.erdos_renyi_lcc(4200, 6, 3)
    if name == "grid9000":        # four lanes per row
        return G.grid_with_deletions(9000, 0.1, 3)
    if name == "star60000":       # a row taken by the block
        return G.star_graph(60000)
    n = int(name[2:])
    return G.barabasi_albert(n, 4, 5)


def _hitting_times(g, w, roots):
    ww = np.ones(g.m) if w is None else w.astype(np.float64)
    A = sp.coo_matrix((np.concatenate([ww, ww]), (np.concatenate([g.src, g.dst]), np.concatenate([g.dst, g.src]))),
                      shape=(g.n, g.n)).tocsr()
    d = np.asarray(A.sum(axis=1)).ravel()
    keep = np.ones(g.n, bool)
    keep[roots] = False
    L = (sp.diags(d) - A).tocsr()[keep][:, keep]
    h = np.zeros(g.n)
    h[keep], info = spl.cg(L, d[keep], rtol=1e-14, maxiter=20000, M=sp.diags(1.0 / d[keep]))
    return h


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("name", ["k2", "ba300", "star4096", "er4096", "er4200", "grid9000", "star60000", "ba200000",
                                  "ba200001"])
def test_solve_in_every_form(name, weighted):
    g = _case(name)
    w = G.uniform_weights(g.m, 0.5, 2.0, 3) if weighted else None
    Gd = P.Graph(g.n, g.src, g.dst, w)
    counts = torch.ones(g.n, dtype=torch.int64, device="cuda")
    a = P.estimate(Gd, counts, 1)
    want = _hitting_times(g, w, [Gd.pivot])
    np.testing.assert_allclose(a["hit"].cpu().numpy(), want, rtol=1e-9, atol=1e-9 * want.max())
    assert float(a["hit"][Gd.pivot]) == 0.0
    b = P.estimate(Gd, counts, 1, stream_ordered=True, max_iter=a["iters"])
    P.workspace_status(b["workspace"])
    assert torch.equal(a["hit"], b["hit"]) and torch.equal(a["rwc"], b["rwc"])
    roots = np.unique([0, g.n // 2])
    if len(roots) < g.n:
        e = P.estimate_group(Gd, roots.astype(np.int32), counts, 1)
        want = _hitting_times(g, w, roots)
        np.testing.assert_allclose(e["hit"].cpu().numpy(), want, rtol=1e-9, atol=1e-9 * want.max())
        assert float(e["hit"][torch.as_tensor(roots)].abs().max()) == 0.0
    if a["iters"] > 1:
        with pytest.raises(P.RWCError) as ei:
            P.estimate(Gd, counts, 1, max_iter=a["iters"] - 1)
        assert ei.value.status == -11
        c = P.estimate(Gd, counts, 1, stream_ordered=True, max_iter=a["iters"] - 1)
        with pytest.raises(P.RWCError):
            P.workspace_status(c["workspace"])


@pytest.mark.parametrize("degree", [63, 64, 65, 200])
def test_longest_row_at_the_block_limit(degree):
    """Four lanes per row take rows of up to 64 entries; a graph with a longer one has them taken by
    the block.  An extra node joined to `degree` nodes of an ER graph, not grounded."""
    g = G.erdos_renyi_lcc(5100, 4, 3)
    to = np.linspace(0, g.n - 1, degree).astype(np.int32)
    g = G.graphs.EdgeList(g.n + 1, np.concatenate([g.src, to]), np.concatenate([g.dst, np.full(degree, g.n, np.int32)]), None)
    assert 2 * g.m <= 6 * g.n and g.n > 4096
    Gd = P.Graph(g.n, g.src, g.dst, None)
    assert Gd.csr.max_degree == degree
    roots = np.array([1, g.n // 2], np.int32)
    e = P.estimate_group(Gd, roots, torch.ones(g.n, dtype=torch.int64, device="cuda"), 1)
    want = _hitting_times(g, None, roots)
    np.testing.assert_allclose(e["hit"].cpu().numpy(), want, rtol=1e-9, atol=1e-9 * want.max())


@pytest.mark.parametrize("n", [4200, 140000, 200001])
def test_sparse_graphs_with_hubs(n):
    """At most three edges a node (four lanes per row) and rows of any length: rows dealt to the blocks, in
    one step and in several, with pairs and with three launches."""
    g = G.barabasi_albert(n, 2, 5)
    Gd = P.Graph(g.n, g.src, g.dst, None)
    assert 2 * g.m <= 6 * g.n and Gd.csr.max_degree > 64
    a = P.estimate(Gd, torch.ones(g.n, dtype=torch.int64, device="cuda"), 1)
    want = _hitting_times(g, None, [Gd.pivot])
    np.testing.assert_allclose(a["hit"].cpu().numpy(), want, rtol=1e-9, atol=1e-9 * want.max())


@pytest.mark.parametrize("a,b", [(300, 4000), (2000, 2200), (20, 40000)])
def test_dense_graphs(a, b):
    """Complete bipartite graphs: rows taken by blocks on one side or both, by more blocks than the rows' own
    lanes fill."""
    g = G.graphs.EdgeList(a + b, np.repeat(np.arange(a), b).astype(np.int32), (a + np.tile(np.arange(b), a)).astype(np.int32), None)
    w = G.uniform_weights(g.m, 0.5, 2.0, 3)
    Gd = P.Graph(g.n, g.src, g.dst, w)
    e = P.estimate(Gd, torch.ones(g.n, dtype=torch.int64, device="cuda"), 1)
    want = _hitting_times(g, w, [Gd.pivot])
    np.testing.assert_allclose(e["hit"].cpu().numpy(), want, rtol=1e-9, atol=1e-9 * want.max())
