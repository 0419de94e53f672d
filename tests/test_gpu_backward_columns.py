"""The adjoint's solve columns at the edges of the blocks of 64 that its directions are stored in (the
product takes two blocks a pass, and none past the last): exact gradients are linear in g, so one of
many targets is the sum of those of its parts.  On a graph large enough that the place of a missing
block lies outside the workspace."""
import numpy as np
import pytest
import torch

import rwcgen as G

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2510_20604_amd")


def _grad(Gd, targets, **kw):
    g = torch.zeros(Gd.n, dtype=torch.float64, device="cuda")
    g[torch.as_tensor(targets, device="cuda")] = 1.0
    return P.backward(Gd, g, tol=1e-12, **kw)["grad_w"]


@pytest.mark.parametrize("parts", [(1, 1), (31, 31), (31, 32), (62, 1), (62, 63), (62, 65), (62, 125), (126, 1), (127, 64)])
def test_gradients_of_parts_add_up(parts):
    g = G.barabasi_albert(200000, 2, 3)
    Gd = P.Graph(g.n, g.src, g.dst, G.uniform_weights(g.m, 0.5, 2.0, 4))
    t = np.random.default_rng(5).choice(g.n, sum(parts), replace=False)
    whole = _grad(Gd, t)
    a, b = _grad(Gd, t[:parts[0]]), _grad(Gd, t[parts[0]:])
    # each within 1e-7 of its largest entry (solves to 1e-12, condition below 1e5)
    bound = 1e-7 * float(whole.abs().max() + a.abs().max() + b.abs().max())
    assert float((a + b - whole).abs().max()) <= bound


@pytest.mark.parametrize("k", [1, 8, 31])
def test_few_probes_on_a_star(k):
    """Few columns on a million nodes: by symmetry every leaf that is no target has the same gradient."""
    g = G.star_graph(1000000)
    Gd = P.Graph(g.n, g.src, g.dst)
    leaf = int(g.dst[17])
    grad = _grad(Gd, [leaf], k=k, seed=3)
    rest = torch.cat([grad[:17], grad[18:]])
    assert torch.isfinite(grad).all()
    assert float(rest.max() - rest.min()) <= 1e-9 * float(rest.abs().max())
