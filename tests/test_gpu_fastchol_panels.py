"""The dense IChol forms panels of 32 columns: sizes at a panel's, a part's (256 rows) and a tile's (64
active rows) edges, no drops (every entry active), and a factor pool
one entry too small, against the oracle bit for bit."""
import numpy as np
import pytest

import rwcgen as G
from test_gpu_fastchol import P, _oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("columns", [31, 32, 33, 63, 64, 65, 95, 97, 127, 129, 255, 257, 287, 289, 321, 513])
@pytest.mark.parametrize("droptol", [0.0, 1e-2])
def test_panel_edges_match_the_oracle(columns, droptol):
    n = columns + 1
    g = G.complete_graph(n) if columns < 100 else G.barabasi_albert(n, 4, columns)
    assert g.n == n
    g = g.with_weights(G.uniform_weights(g.m, 0.5, 2.0, columns))
    Gd = P.Graph(g.n, g.src, g.dst, g.w)
    tau, fnz, snz = _oracle(g, Gd.pivot, droptol, 8.0, 8, 1e-3)
    r = P.fastchol(Gd, droptol=droptol, window=8.0, zeta=8, factor_capacity=fnz, inverse_capacity=snz, method="dense")
    assert (r["factor_entries"], r["inverse_entries"]) == (fnz, snz)
    np.testing.assert_array_equal(r["tau"].cpu().numpy(), tau)
    if fnz - 1 >= columns:
        with pytest.raises(P.RWCError) as ei:
            P.fastchol(Gd, droptol=droptol, window=8.0, zeta=8, factor_capacity=fnz - 1, inverse_capacity=snz, method="dense")
        assert ei.value.status == -7


@pytest.mark.parametrize("name,window,zeta,eps_p", [
    ("ba", 16.0, 12, 1e-3), ("ba", 16.5, 12, 1e-3), ("ba", 33.0, 12, 1e-3),   # windows to 32 columns, to 33, all above
    ("ba", 16.0, 63, 1e-3), ("ba", 16.0, 64, 1e-9), ("ba", 16.0, 70, 1e-3),   # columns of 64 entries and more
    ("ba", 16.0, 126, 0.0), ("ba", 16.0, 200, 0.0),                           # 128 distinct rows and more
    ("clique", 16.0, 10, 1e-3), ("cycle", 16.0, 0, 0.5), ("star", 16.0, 2, 1e-3)])   # equal magnitudes
def test_inverse_columns_match_the_oracle(name, window, zeta, eps_p):
    """The inverse's columns in LDS and in the workspace, and both in one run, bit for bit."""
    g = {"ba": lambda: G.barabasi_albert(700, 4, 3), "clique": lambda: G.complete_graph(90),
         "cycle": lambda: G.cycle_graph(200), "star": lambda: G.star_graph(300)}[name]()
    if name == "ba":
        g = g.with_weights(G.uniform_weights(g.m, 0.5, 2.0, 5))
    Gd = P.Graph(g.n, g.src, g.dst, g.w)
    tau, fnz, snz = _oracle(g, Gd.pivot, 1e-4, window, zeta, eps_p)
    r = P.fastchol(Gd, droptol=1e-4, window=window, zeta=zeta, eps_p=eps_p, factor_capacity=fnz, inverse_capacity=snz)
    assert (r["factor_entries"], r["inverse_entries"]) == (fnz, snz)
    np.testing.assert_array_equal(r["tau"].cpu().numpy(), tau)


@pytest.mark.parametrize("columns", [32, 33, 699])
@pytest.mark.parametrize("window,zeta", [(32.0, 3), (32.9, 12), (33.0, 12), (64.0, 20), (64.5, 20), (150.0, 40)])
def test_long_windows_match_the_oracle(columns, window, zeta):
    """Windows that no column in LDS serves (33 and more), the longest (over 64), and matrices of no more
    columns than the windows in LDS hold, where they still do."""
    g = G.complete_graph(columns + 1) if columns < 100 else G.barabasi_albert(columns + 1, 4, 3)
    g = g.with_weights(G.uniform_weights(g.m, 0.5, 2.0, 5))
    Gd = P.Graph(g.n, g.src, g.dst, g.w)
    tau, fnz, snz = _oracle(g, Gd.pivot, 1e-4, window, zeta, 1e-3)
    r = P.fastchol(Gd, droptol=1e-4, window=window, zeta=zeta, eps_p=1e-3, factor_capacity=fnz, inverse_capacity=snz)
    assert (r["factor_entries"], r["inverse_entries"]) == (fnz, snz)
    np.testing.assert_array_equal(r["tau"].cpu().numpy(), tau)


def test_columns_over_the_lds_limit_with_short_windows():
    """A ring of cliques: columns of the inverse of up to a thousand rows in windows of 12."""
    a, b = np.triu_indices(16, 1)
    c = np.arange(70)
    src = np.concatenate([(a[None] + 16 * c[:, None]).ravel(), 16 * c])
    dst = np.concatenate([(b[None] + 16 * c[:, None]).ravel(), 16 * ((c + 1) % 70) + 1])
    g = G.graphs.EdgeList(16 * 70, src.astype(np.int32), dst.astype(np.int32), None)
    g = g.with_weights(G.uniform_weights(g.m, 0.5, 2.0, 5))
    Gd = P.Graph(g.n, g.src, g.dst, g.w)
    tau, fnz, snz = _oracle(g, Gd.pivot, 1e-4, 12.0, 12, 1e-6)
    assert snz > 400 * g.n      # columns of hundreds of entries
    r = P.fastchol(Gd, droptol=1e-4, window=12.0, zeta=12, eps_p=1e-6, factor_capacity=fnz, inverse_capacity=snz)
    assert (r["factor_entries"], r["inverse_entries"]) == (fnz, snz)
    np.testing.assert_array_equal(r["tau"].cpu().numpy(), tau)
