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
