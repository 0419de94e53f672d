"""The autotuners against the plan a call takes when it leaves the plan open.  Where that pops cycles in
rounds the tuned call must not be a slower one: it pops them too (measured 2 to 6 times faster than any
plan of walkers on these graphs), with the same forest."""
import pytest
import torch

import rwcgen as G

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2510_20604_amd")

SCHEDULE = ("path_ring", "bfs_starts", "lds_state")


def _same(a, b):
    for key in ("counts", "counts_sq", "tree_hash", "total_steps"):
        assert torch.equal(a[key], b[key]), key


@pytest.mark.parametrize("name,kernel", [("er", "cycle_pop"), ("ba", "cycle_pop"), ("mesh", "mesh_pop"), ("big", None)])
def test_single_graph(name, kernel):
    g = {"er": lambda: G.erdos_renyi_lcc(1000, 8, 1), "ba": lambda: G.barabasi_albert(9000, 5, 1),
         "mesh": lambda: G.grid_with_deletions(5000, 0.1, 1), "big": lambda: G.barabasi_albert(30100, 4, 1)}[name]()
    Gd = P.Graph(g.n, g.src, g.dst)
    P._lib.lib().rwc_autotune_clear_cache()
    t = P.autotune(Gd, 300, 7)
    assert t["walkers_per_tree"] in (1, 8, 16, 32, 64) and t["trees_in_flight"] >= 1
    assert (t["lds_state"] == "pop") == (kernel is not None)
    s = P.sample_forests(Gd, 300, 7, walkers_per_tree=t["walkers_per_tree"], trees_in_flight=t["trees_in_flight"],
                         starts=t["starts"], **{k: t[k] for k in SCHEDULE})
    _same(s, P.sample_forests(Gd, 300, 7, lds_state=False))
    if kernel:
        assert s["walk_kernel"] == kernel
        # no room for the open plan's sums and counts: a plan of walkers
        P._lib.lib().rwc_autotune_clear_cache()
        assert P.autotune(Gd, 300, 7, budget_bytes=g.n * 8 * 64)["lds_state"] != "pop"
    else:
        assert s["walk_kernel"].startswith("wilson")


def test_batch():
    graphs = [P.Graph(g.n, g.src, g.dst, g.w) for g in G.batch_mix(8, 500, 4000, seed=47)]
    P._lib.lib().rwc_autotune_clear_cache()
    t = P.autotune_batch(graphs, 96, 13)
    assert t["candidates"] == 17 and t["lds_state"] == "pop"
    s = P.sample_forests(graphs, 96, 13, persistent=True, walkers_per_graph=t["walkers_per_graph"],
                         **{k: t[k] for k in SCHEDULE})
    assert s["walk_kernel"] in ("cycle_pop", "mesh_pop")
    _same(s, P.sample_forests(graphs, 96, 13, lds_state=False))
    graphs.append(P.Graph(*(lambda g: (g.n, g.src, g.dst))(G.barabasi_albert(30100, 4, 1))))   # too large for the rounds
    assert P.autotune_batch(graphs, 96, 13)["lds_state"] != "pop"
