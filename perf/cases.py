"""Timed cases over the framework's public entry points, for comparing two versions of it.

listed() covers what a program does with the framework: random walk centrality end to end on
small and large graphs, sampling on a graph that is kept, batches, meshes, the CSR build, the
gradient with respect to the edge weights, groups of nodes and FastChol.  draw() gives further
sizes of the same kinds.  A case's topology is fixed by its own fields (the generators of
rwcgen); the seed decides the edge weights, the sampling keys and the upstream gradients.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2510_20604_amd as P
import rwcgen


def listed():
    return [
        # one call on a graph of a few hundred nodes: launches and host work count, not bandwidth
        dict(name="call_er300", kind="call", graph="er", n=300, deg=8, weighted=True, l=200),
        # the small benchmark graph, whole pipeline: trees that fit the LDS
        dict(name="rwc_er1000", kind="rwc", graph="er", n=1000, deg=8, weighted=False, l=2000, strata=False),
        # a middle-sized heavy-tailed graph with stratified stack entries and standard errors
        dict(name="rwc_ba20k_strata", kind="rwc", graph="ba", n=20000, deg=5, weighted=False, l=2000, strata=True),
        # a road-like mesh: long walks, many solver iterations, a deep breadth-first order
        dict(name="rwc_grid97k", kind="rwc", graph="grid", n=97000, deg=0, weighted=True, l=300, strata=False),
        # sampling with a kept graph and workspace: a million-node network, part of its trees
        dict(name="sample_ba1m", kind="sample", graph="ba", n=1000000, deg=5, weighted=False, l=2000),
        # the headline step at a quarter of its size: CSR build, trees, pivot solve, adjoint
        dict(name="step_rmat21", kind="step", graph="rmat", n=1 << 21, deg=5, weighted=True, l=2000, targets=1000, k=64),
        # many graphs of uneven size in one persistent, captured launch
        dict(name="batch_64", kind="batch", graphs=64, n_lo=1000, n=20000, l=200),
        # the CSR build alone, weighted
        dict(name="build_ba1m", kind="build", graph="ba", n=1000000, deg=5, weighted=True),
        # forests rooted at the 16 largest hubs and the marginal of every further member
        dict(name="group_ba200k", kind="group", graph="ba", n=200000, deg=5, weighted=False, l=1000, roots=16),
        # the gradient for 100 targets through 64 probes
        dict(name="grad_ba100k", kind="grad", graph="ba", n=100000, deg=4, weighted=True, targets=100, k=64),
        # a training step on a small weighted graph: forward estimate and weight gradient
        dict(name="train_ba2k", kind="train", graph="ba", n=2000, deg=4, weighted=True, l=500, k=16),
        # FastChol with the paper's parameters
        dict(name="fastchol_ba5k", kind="fastchol", graph="ba", n=5000, deg=5, weighted=True),
    ]


def _spread(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["call", "rwc", "rwc", "grid", "sample", "sample", "step", "batch", "build", "group", "grad",
                       "train", "fastchol"])
    deg = rng.randint(2, 8)
    weighted = rng.random() < 0.5
    if kind == "call":
        return dict(kind="call", graph=rng.choice(["er", "ba"]), n=_spread(rng, 100, 2000), deg=max(deg, 4),
                    weighted=weighted, l=_spread(rng, 50, 1000))
    if kind == "rwc":
        n = _spread(rng, 500, 100000)
        return dict(kind="rwc", graph=rng.choice(["er", "ba"]), n=n, deg=max(deg, 4), weighted=weighted,
                    l=_spread(rng, 100, 4000), strata=rng.random() < 0.3)
    if kind == "grid":
        n = _spread(rng, 500, 97000)
        return dict(kind="rwc", graph="grid", n=n, deg=0, weighted=weighted, l=_spread(rng, 50, 300), strata=False)
    if kind == "sample":
        n = _spread(rng, 20000, 1000000)
        return dict(kind="sample", graph=rng.choice(["ba", "rmat"]), n=n, deg=min(deg, 6), weighted=weighted,
                    l=_spread(rng, 200, 2000))
    if kind == "step":
        n = _spread(rng, 4000, 300000)
        return dict(kind="step", graph=rng.choice(["ba", "rmat"]), n=n, deg=min(deg, 6), weighted=True,
                    l=_spread(rng, 200, 2000), targets=_spread(rng, 10, 1000), k=rng.choice([16, 32, 48, 64]))
    if kind == "batch":
        return dict(kind="batch", graphs=rng.randint(8, 64), n_lo=300, n=_spread(rng, 1500, 20000),
                    l=_spread(rng, 50, 200))
    if kind == "build":
        return dict(kind="build", graph=rng.choice(["er", "ba", "rmat", "grid"]), n=_spread(rng, 1000, 1000000),
                    deg=max(3, min(deg, 6)), weighted=weighted)
    if kind == "group":
        return dict(kind="group", graph="ba", n=_spread(rng, 2000, 200000), deg=min(deg, 6), weighted=weighted,
                    l=_spread(rng, 100, 1000), roots=rng.randint(2, 32))
    if kind == "grad":
        return dict(kind="grad", graph=rng.choice(["ba", "rmat"]), n=_spread(rng, 2000, 100000), deg=min(deg, 6),
                    weighted=weighted, targets=_spread(rng, 5, 100), k=rng.choice([0, 8, 16, 32, 64]))
    if kind == "train":
        return dict(kind="train", graph=rng.choice(["er", "ba"]), n=_spread(rng, 300, 10000), deg=max(deg, 4),
                    weighted=True, l=_spread(rng, 100, 1000), k=rng.choice([4, 8, 16, 32]))
    return dict(kind="fastchol", graph=rng.choice(["er", "ba"]) if rng.random() < 0.5 else "ba",
                n=_spread(rng, 300, 5000), deg=min(max(deg, 4), 6), weighted=True)


# -- inputs ---------------------------------------------------------------------------------
@functools.lru_cache(maxsize=4)
def _topology(graph, n, deg):
    seed = 1000 + n % 9973
    if graph == "er":
        return rwcgen.erdos_renyi_lcc(n, deg, seed)
    if graph == "ba":
        return rwcgen.barabasi_albert(n, deg, seed)
    if graph == "grid":
        return rwcgen.grid_with_deletions(n, 0.1, seed)
    return rwcgen.rmat_lcc(max(4, round(math.log2(n))), deg, 0.57, 0.19, 0.19, seed)


@functools.lru_cache(maxsize=2)
def _batch_topology(graphs, n_lo, n):
    return rwcgen.batch_mix(graphs, n_lo, n, 1003)


def _weights(m, lo, hi, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return torch.rand(m, generator=gen, device="cuda", dtype=torch.float32) * (hi - lo) + lo


def _edges(case, seed):
    g = _topology(case["graph"], case["n"], case["deg"])
    lo, hi = (1.0, 4.0) if case["graph"] == "rmat" else (0.5, 2.0)
    return dict(n=g.n, src=torch.from_numpy(g.src.astype(np.int32)).cuda(),
                dst=torch.from_numpy(g.dst.astype(np.int32)).cuda(),
                w=_weights(g.m, lo, hi, seed) if case["weighted"] else None, seed=100003 * (seed + 1))


def _targets(n, count, seed):
    """g = 1 at `count` nodes drawn uniformly: the sum of their centralities is differentiated."""
    gen = torch.Generator()
    gen.manual_seed(seed + 17)
    g = torch.zeros(n, dtype=torch.float64)
    g[torch.randperm(n, generator=gen)[:min(count, n)]] = 1.0
    return g.cuda()


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        gl = _batch_topology(case["graphs"], case["n_lo"], case["n"])
        graphs = [P.Graph(g.n, g.src, g.dst, _weights(g.m, 0.5, 2.0, seed + 31 * i), "cuda") for i, g in enumerate(gl)]
        return dict(case=case, graphs=graphs, seed=100003 * (seed + 1), out=None)
    s = dict(case=case, **_edges(case, seed))
    if kind in ("sample", "group", "grad", "fastchol"):
        s["G"] = P.Graph(s["n"], s["src"], s["dst"], s["w"], "cuda")
    if kind in ("grad", "step"):
        s["g"] = _targets(s["n"], case["targets"], seed)
    if kind == "train":
        gen = torch.Generator(device="cuda")
        gen.manual_seed(seed + 5)
        s["g"] = torch.randn(s["n"], generator=gen, device="cuda", dtype=torch.float64) / s["n"]
        s["w"].requires_grad_(True)
    if kind == "group":
        deg = torch.zeros(s["n"], dtype=torch.int64, device="cuda")
        one = torch.ones_like(s["src"], dtype=torch.int64)
        deg.index_add_(0, s["src"].long(), one).index_add_(0, s["dst"].long(), one)
        s["roots"] = torch.argsort(deg, descending=True, stable=True)[:case["roots"]].to(torch.int32)
    s["ws"] = None
    return s


# -- one pass -------------------------------------------------------------------------------
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "call":
        return P.random_walk_centrality(s["n"], s["src"], s["dst"], s["w"], l=case["l"], seed=s["seed"])
    if kind == "rwc":
        G = P.Graph(s["n"], s["src"], s["dst"], s["w"], "cuda")
        f = P.sample_forests(G, case["l"], s["seed"], want_hash=False, strata=case["l"] if case["strata"] else 0)
        e = P.estimate(G, f["counts"], case["l"], counts_sq=f["counts_sq"], want_stderr=True)
        return {"counts": f["counts"], "counts_sq": f["counts_sq"], "steps": f["total_steps"], "rwc": e["rwc"],
                "hit": e["hit"], "stderr": e["stderr"]}
    if kind == "sample":
        f = P.sample_forests(s["G"], case["l"], s["seed"], want_hash=False, workspace=s["ws"])
        s["ws"] = f["workspace"]
        return {"counts": f["counts"], "counts_sq": f["counts_sq"], "steps": f["total_steps"]}
    if kind == "batch":
        f = P.sample_forests(s["graphs"], case["l"], s["seed"], persistent=True, capture=True, want_sq=False,
                             want_hash=False, workspace=s["out"]["workspace"] if s["out"] else None, out=s["out"])
        s["out"] = f
        return {"counts": f["counts"], "steps": f["total_steps"]}
    if kind == "build":
        G = P.Graph(s["n"], s["src"], s["dst"], s["w"], "cuda")
        r = {"row_ptr": G.row_ptr(), "col": G.col(), "weight": G.weight(), "edge_id": G.edge_id(),
             "strength": G.strength(), "node_id": G.node_id(), "component": G.component(), "rec": G.rec(),
             "pivot": G.pivot, "vol": G.vol}
        if s["w"] is not None:
            r["cdf"] = G.cdf()
        return r
    if kind == "step":
        G = P.Graph(s["n"], s["src"], s["dst"], s["w"], "cuda")
        f = P.sample_forests(G, case["l"], s["seed"], persistent=True, want_hash=False, workspace=s["ws"])
        s["ws"] = f["workspace"]
        e = P.estimate(G, f["counts"], case["l"], counts_sq=f["counts_sq"], want_stderr=True)
        b = P.backward(G, s["g"], k=case["k"], seed=s["seed"] + 1)
        return {"counts": f["counts"], "counts_sq": f["counts_sq"], "steps": f["total_steps"], "rwc": e["rwc"],
                "hit": e["hit"], "stderr": e["stderr"], "grad": b["grad_w"]}
    if kind == "group":
        f = P.sample_forests(s["G"], case["l"], s["seed"], roots=s["roots"], want_sq=False, want_hash=False,
                             workspace=s["ws"])
        s["ws"] = f["workspace"]
        e = P.estimate_group(s["G"], s["roots"], f["counts"], case["l"])
        return {"counts": f["counts"], "steps": f["total_steps"], "group_rwc": e["group_rwc"],
                "marginal": e["marginal"], "hit": e["hit"]}
    if kind == "grad":
        return P.backward(s["G"], s["g"], k=case["k"], seed=s["seed"] + 1)["grad_w"]
    if kind == "train":
        rwc = P.RWCFunction.apply(s["w"], s["n"], s["src"], s["dst"], case["l"], s["seed"], case["k"])
        gw, = torch.autograd.grad(rwc, s["w"], s["g"])
        return {"rwc": rwc.detach(), "grad": gw}
    width = math.ceil(math.log2(s["n"]))
    tau = P.fastchol(s["G"], window=width, zeta=width)["tau"]
    e = P.estimate_diag(s["G"], tau)
    return {"tau": tau, "rwc": e["rwc"], "hit": e["hit"]}


# -- what a pass cannot do without ----------------------------------------------------------
# Random-neighbour steps per node and tree, as measured: the walk's own data is 28 bytes a step
# (row bounds, the chosen entry, the next state word read, the own one written), 16 bytes per
# attached node and 8 bytes per node for the scan of start nodes.
_STEPS = {"er": 1.3, "ba": 1.15, "rmat": 1.05, "grid": 14.0}


def _tree_bytes(graph, n, l, weighted):
    return l * n * (_STEPS[graph] * (36.0 if weighted else 28.0) + 24.0)


def _solve_bytes(n, m, columns, iterations):
    return iterations * (24.0 * m + 40.0 * n * columns), iterations * columns * (4.0 * m + 12.0 * n)


def _iterations(graph, n):
    return 4.0 * math.sqrt(n) if graph == "grid" else 40.0


def work(case):
    kind = case["kind"]
    if kind == "batch":
        gl = _batch_topology(case["graphs"], case["n_lo"], case["n"])
        half = len(gl) // 2
        b = sum(_tree_bytes("ba" if i < half else "grid", g.n, case["l"], True) for i, g in enumerate(gl))
        return {"bytes": b, "flops": 0.0}
    g = _topology(case["graph"], case["n"], case["deg"])
    n, m, graph = g.n, g.m, case["graph"]
    it = _iterations(graph, n)
    b = f = 0.0
    if kind in ("call", "rwc", "step", "build", "train"):
        b += m * (8.0 + 4.0 * case["weighted"]) + 2 * m * (12.0 + 8.0 * case["weighted"]) + 100.0 * n
    if kind in ("call", "rwc", "step", "sample", "group", "train"):
        b += _tree_bytes(graph, n, case["l"], case["weighted"]) + 16.0 * n
    if kind in ("call", "rwc", "step", "group", "train", "fastchol"):
        sb, sf = _solve_bytes(n, m, 1, it)
        b, f = b + sb + 24.0 * n, f + sf
    if kind in ("grad", "step", "train"):
        columns = 2 + (case["k"] if kind != "train" else 2 * case["k"])
        if kind == "grad" and case["k"] == 0:
            columns = 2 + case["targets"]
        sb, sf = _solve_bytes(n, m, columns, it)
        b, f = b + sb + 8.0 * m, f + sf + 6.0 * m * columns
    if kind == "fastchol":
        # the factor keeps a few hundred entries per column; each pair of them is updated once
        kept = min(350.0, n / 3.0)
        b, f = b + 12.0 * n * kept, f + n * kept * kept
    return {"bytes": b, "flops": f}


# -- the same values in plain torch, 64 bits -------------------------------------------------
def _laplacian(s):
    """Weighted degrees and the adjacency as a sparse float64 matrix."""
    n = s["n"]
    a, b = s["src"].long(), s["dst"].long()
    w = torch.ones(a.numel(), dtype=torch.float64, device=a.device) if s["w"] is None else s["w"].detach().double()
    d = torch.zeros(n, dtype=torch.float64, device=a.device).index_add_(0, a, w).index_add_(0, b, w)
    A = torch.sparse_coo_tensor(torch.stack([torch.cat([a, b]), torch.cat([b, a])]), torch.cat([w, w]), (n, n))
    return a, b, d, A.coalesce().to_sparse_csr()


def _solve(A, d, rhs, keep, tol=1e-14, most=6000):
    """Jacobi-preconditioned CG on the Laplacian restricted to the nodes `keep`; rhs [n, c]."""
    keep = keep.double()[:, None]
    b = rhs * keep
    x = torch.zeros_like(b)
    r = b.clone()
    z = r / d[:, None]
    p = z.clone()
    rz = (r * z).sum(0)
    stop = tol * b.norm(dim=0)
    for i in range(most):
        q = (d[:, None] * p - A @ p) * keep
        pq = (p * q).sum(0)
        alpha = torch.where(pq > 0, rz / pq, torch.zeros_like(rz))
        x += alpha * p
        r -= alpha * q
        if i % 8 == 7 and bool((r.norm(dim=0) <= stop).all()):
            break
        z = r / d[:, None]
        new = (r * z).sum(0)
        p = z + torch.where(rz > 0, new / rz, torch.zeros_like(rz)) * p
        rz = new
    return x


def _philox_bit(key, counters, node):
    """Bit 0 of Philox4x32-10's first word on the counters (probe, node, 0, 2^32 - 1)."""
    lo = np.uint64(0xFFFFFFFF)
    c = [counters.astype(np.uint64), node.astype(np.uint64), np.zeros_like(node, dtype=np.uint64),
         np.full(node.shape, 0xFFFFFFFF, dtype=np.uint64)]
    k0, k1 = key & 0xFFFFFFFF, (key >> 32) & 0xFFFFFFFF
    for _ in range(10):
        p0, p1 = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
        c = [((p1 >> np.uint64(32)) ^ c[1] ^ np.uint64(k0)) & lo, p1 & lo,
             ((p0 >> np.uint64(32)) ^ c[3] ^ np.uint64(k1)) & lo, p0 & lo]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return (c[0] & np.uint64(1)).astype(np.float64)


def _gradient(s, k, key):
    """d(sum_j g_j RWC_j)/dw_e through L^+: see the adjoint's formula in the C header."""
    a, b, d, A = _laplacian(s)
    n, g = s["n"], s["g"]
    dev = g.device
    support = torch.nonzero(g).flatten()
    root = g.abs().sqrt()
    cols, coef = [g, d], []
    for cls in (0, 1):
        sel = support[g[support] > 0] if cls == 0 else support[g[support] < 0]
        if sel.numel() == 0:
            continue
        if k == 0:
            for t in sel.tolist():
                y = torch.zeros(n, dtype=torch.float64, device=dev)
                y[t] = root[t]
                cols.append(y)
                coef.append(1.0 if cls == 0 else -1.0)
            continue
        for i in range(k):
            node = sel.cpu().numpy()
            bit = _philox_bit(key, np.full(node.shape, cls * k + i), node)
            y = torch.zeros(n, dtype=torch.float64, device=dev)
            y[sel] = torch.from_numpy(1.0 - 2.0 * bit).to(dev) * root[sel]
            cols.append(y)
            coef.append((1.0 if cls == 0 else -1.0) / k)
    Y = torch.stack(cols, 1)
    del cols
    keep = torch.ones(n, dtype=torch.bool, device=dev)
    keep[torch.argmax(d)] = False
    X = _solve(A, d, Y - Y.mean(0), keep, tol=1e-13, most=1500)
    X -= X.mean(0)
    vol, G = d.sum(), g.sum()
    Q = torch.zeros(a.numel(), dtype=torch.float64, device=dev)
    tr = torch.zeros((), dtype=torch.float64, device=dev)
    for i, c in enumerate(coef):
        z = X[:, 2 + i].contiguous()
        Q += c * (z[a] - z[b]) ** 2
        tr += c * (Y[:, 2 + i] * z).sum()
    XA, XB = X[:, 0].contiguous(), X[:, 1].contiguous()
    DA, SA, DB, SB = XA[a] - XA[b], XA[a] + XA[b], XB[a] - XB[b], XB[a] + XB[b]
    return 2 * tr - vol * Q + 2 * DA * DB - 2 * SA + G * ((2 * SB - DB * DB) / vol - 2 * (d * XB).sum() / vol ** 2)


def exact(case, seed):
    """The outputs that plain linear algebra defines: hitting times, the group's centrality and
    gradients.  Counts of sampled trees, what is made from them, and FastChol's diagonal (an
    incomplete factor, column by column) have no such value here."""
    kind = case["kind"]
    if kind in ("call", "sample", "batch", "build"):
        return None
    s = _edges(case, seed)
    if kind in ("grad", "step"):
        s["g"] = _targets(s["n"], case["targets"], seed)
    if kind == "train":
        gen = torch.Generator(device="cuda")
        gen.manual_seed(seed + 5)
        s["g"] = torch.randn(s["n"], generator=gen, device="cuda", dtype=torch.float64) / s["n"]
        return {"rwc": None, "grad": _gradient(s, case["k"], 0)}
    if kind == "grad":
        return _gradient(s, case["k"], s["seed"] + 1)
    _, _, d, A = _laplacian(s)
    keep = torch.ones(s["n"], dtype=torch.bool, device=d.device)
    if kind == "group":
        s = prepare(case, seed)
        keep[s["roots"].long()] = False
    else:
        # the pivot: the largest weighted degree in units of 2^-24, ties to the smallest id
        fixed = torch.round(d * 2.0 ** 24)
        keep[torch.nonzero(fixed == fixed.max()).flatten()[0]] = False
    hit = _solve(A, d, d[:, None], keep)[:, 0]
    if kind == "group":
        return {"counts": None, "steps": None, "group_rwc": ((d * hit).sum() / d.sum()).reshape(1), "marginal": None,
                "hit": hit}
    if kind == "fastchol":
        return {"tau": None, "rwc": None, "hit": hit}
    r = {"counts": None, "counts_sq": None, "steps": None, "rwc": None, "hit": hit, "stderr": None}
    if kind == "step":
        r["grad"] = _gradient(s, case["k"], s["seed"] + 1)
    return r
