"""Performance cases: the work a user of this package has it do, through its
public entry points, over the sizes the package's own tests and benchmark use.

Six kinds of case:
  zoom    one interactive zoom step of the multi-level view: level-l DPPR of a
          supernode's k children by Tau-Push, PDist, a short layout;
  level   level-l DPPR of the top supernode of a large graph (Group
          Forward-Push);
  ppr     multi-source PPR/DPPR of one graph, to a residual tolerance, and
          PDist among the sources (and a short layout, where asked for);
  layout  Jacobi sweeps of one layout, or one exact majorization step;
  grad    one training step: gradients of the layout stress with respect to
          every edge weight and every coordinate;
  batch   the captured pipeline over many ragged subgraphs (all-pairs PPR,
          PDist, layout).

Graphs are Erdos-Renyi, Chung-Lu and stochastic block models, the families the
package's tests and benchmark draw from.  Layouts start from U[-1, 1]^2.  The
layouts run a few tens of sweeps: the objective is not convex, and a longer
run from a random start can amplify a difference of one rounding without
bound, so that nothing could be said about its result.
"""
import math
import types

import numpy as np
import torch

from paper_2112_14944_amd import autograd, ops

ALPHA = 0.15
DEV = "cuda"


# ------------------------------------------------------------------- cases

def listed():
    return [
        # A user clicks a supernode of a 20000-node graph: its k = 25 children
        # are placed anew.  The smallest call; its latency is what the user sees.
        {"name": "zoom_k25", "kind": "zoom", "n": 20000, "gamma": 2.5, "degree": 20.0, "k": 25, "sweeps": 50},
        # A small graph drawn from scratch: all pairs to 1e-10, PDist, layout.
        {"name": "draw_er500", "kind": "ppr", "graph": "er", "n": 500, "degree": 8.0, "sources": 500,
         "tol": 1e-10, "sweeps": 50},
        # The largest graph of the all-on-chip range, all pairs.
        {"name": "ppr_sbm2048", "kind": "ppr", "graph": "sbm", "n": 2048, "blocks": 8, "p_in": 0.2, "p_out": 0.01,
         "sources": 2048, "tol": 1e-6, "sweeps": 0},
        # A query: the PDist of a few dozen chosen nodes of a mid-size graph.
        {"name": "query_cl20000", "kind": "ppr", "graph": "cl", "n": 20000, "gamma": 2.5, "degree": 20.0,
         "sources": 48, "tol": 1e-7, "sweeps": 0},
        # All pairs of the same graph, the way a single-level drawing of it needs them.
        {"name": "ppr_cl20000", "kind": "ppr", "graph": "cl", "n": 20000, "gamma": 2.5, "degree": 20.0,
         "sources": 20000, "tol": 1e-7, "sweeps": 0},
        # A query on a graph whose iterate lives in HBM.
        {"name": "query_cl1e6", "kind": "ppr", "graph": "cl", "n": 1000000, "gamma": 2.2, "degree": 30.0,
         "sources": 64, "tol": 1e-6, "sweeps": 0},
        # Top level of a 10^6-node hierarchy: 25 supernodes of 40000 leaves.
        {"name": "level_cl1e6", "kind": "level", "n": 1000000, "gamma": 2.2, "degree": 30.0, "k": 25},
        # An ordinary single layout (odd size), and one exact step of a larger one.
        {"name": "layout_k1999", "kind": "layout", "k": 1999, "sweeps": 50, "exact": False},
        {"name": "exact_k4096", "kind": "layout", "k": 4096, "sweeps": 1, "exact": True},
        # Training steps: a small graph, and the largest the tests differentiate.
        {"name": "grad_sbm1000", "kind": "grad", "n": 1000, "blocks": 8, "degree": 24.0, "T": 100},
        {"name": "grad_sbm8192", "kind": "grad", "n": 8192, "blocks": 32, "degree": 24.0, "T": 100},
        # A server's batch of subgraphs, 32 to 2048 nodes, one replay of the captured pipeline.
        {"name": "batch_512", "kind": "batch", "graphs": 512, "n_lo": 32, "n_hi": 2048, "p_in": 0.2, "p_out": 0.01,
         "tol": 1e-6, "sweeps": 30},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["zoom", "ppr", "ppr", "ppr", "query", "level", "layout", "layout", "grad", "batch", "batch"])
    if kind == "zoom":
        return {"kind": "zoom", "n": _log(rng, 2000, 60000), "gamma": round(rng.uniform(2.2, 2.8), 2),
                "degree": round(rng.uniform(8, 30), 1), "k": rng.randint(8, 40), "sweeps": rng.randint(20, 50)}
    if kind == "ppr":  # all pairs
        graph = rng.choice(["er", "sbm", "cl"])
        case = {"kind": "ppr", "graph": graph, "n": _log(rng, 33, 2304 if graph == "sbm" else 12000),
                "tol": rng.choice([1e-6, 1e-7, 1e-10])}
        case["sources"] = case["n"]
        if graph == "sbm":
            case |= {"blocks": rng.randint(4, 16), "p_in": 0.2, "p_out": 0.01}
        else:
            case["degree"] = round(rng.uniform(6, 30), 1)
        if graph == "cl":
            case["gamma"] = round(rng.uniform(2.3, 2.8), 2)
        case["sweeps"] = rng.choice([0, 30])
        return case
    if kind == "query":
        n = _log(rng, 1000, 1000000)
        return {"kind": "ppr", "graph": "cl", "n": n, "gamma": round(rng.uniform(2.2, 2.8), 2),
                "degree": round(rng.uniform(8, 30), 1), "sources": _log(rng, 1, 256 if n < 200000 else 64),
                "tol": rng.choice([1e-6, 1e-7]), "sweeps": 0}
    if kind == "level":
        return {"kind": "level", "n": _log(rng, 50000, 1000000), "gamma": round(rng.uniform(2.2, 2.6), 2),
                "degree": round(rng.uniform(10, 30), 1), "k": rng.randint(10, 40)}
    if kind == "layout":
        exact = rng.random() < 0.4
        return {"kind": "layout", "k": _log(rng, 25, 8000), "sweeps": 1 if exact else rng.randint(10, 50),
                "exact": exact}
    if kind == "grad":
        return {"kind": "grad", "n": _log(rng, 300, 6000), "blocks": rng.randint(4, 24),
                "degree": round(rng.uniform(12, 30), 1), "T": 100}
    return {"kind": "batch", "graphs": _log(rng, 8, 384), "n_lo": 32, "n_hi": rng.choice([300, 1000, 2048]),
            "p_in": 0.2, "p_out": 0.01, "tol": 1e-6, "sweeps": rng.randint(10, 30)}


# ------------------------------------------------------------------ inputs

def _gen(seed, salt=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * seed + salt)
    return g


def _csr_from_pairs(n, a, b):
    """Symmetric CSR (sorted rows, no loops, no repeats) of undirected pairs.
    Returns row_ptr int32[n+1], rows int64[nnz], cols int64[nnz]."""
    keep = a != b
    a, b = a[keep], b[keep]
    key = torch.unique(torch.minimum(a, b) * n + torch.maximum(a, b))
    lo, hi = key // n, key % n
    key = torch.sort(torch.cat([lo * n + hi, hi * n + lo])).values
    rows, cols = key // n, key % n
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    row_ptr[1:] = torch.cumsum(torch.bincount(rows, minlength=n), 0)
    return row_ptr.to(torch.int32), rows, cols


def _chung_lu(n, gamma, degree, gen):
    w = torch.arange(1, n + 1, dtype=torch.float64, device=DEV) ** (-1.0 / (gamma - 1.0))
    w *= degree / w.mean()
    for _ in range(30):
        w = torch.clamp(w, max=math.sqrt(float(w.sum())))
        w *= degree / w.mean()
    w = torch.clamp(w, max=math.sqrt(float(w.sum())))
    cdf = torch.cumsum(w / w.sum(), 0)
    cdf[-1] = 1.0
    m = int(float(w.sum()) / 2)
    ends = torch.rand((2, m), dtype=torch.float64, device=DEV, generator=gen)
    ends = torch.searchsorted(cdf, ends).clamp(max=n - 1)
    return _csr_from_pairs(n, ends[0], ends[1])


def _uniform_pairs(n, degree, gen):
    """n degree / 2 uniform pairs (the few repeats collapse)."""
    e = torch.randint(0, n, (2, int(round(n * degree / 2))), device=DEV, generator=gen)
    return e[0], e[1]


def _block_sizes(n, blocks):
    blocks = min(blocks, n)
    return [n // blocks + (1 if i < n % blocks else 0) for i in range(blocks)]


def _sbm_dense(n, blocks, p_in, p_out, gen):
    """Every pair of an n-node block model drawn by itself."""
    sizes = torch.tensor(_block_sizes(n, blocks), device=DEV)
    label = torch.repeat_interleave(torch.arange(len(sizes), device=DEV), sizes)
    p = torch.where(label[:, None] == label[None, :], p_in, p_out)
    hit = torch.triu(torch.rand((n, n), device=DEV, generator=gen) < p, diagonal=1)
    a, b = torch.nonzero(hit, as_tuple=True)
    return _csr_from_pairs(n, a, b)


def _sbm_edges(n, blocks, degree, gen):
    """Block model with exactly n degree / 2 edges, about four fifths of them
    inside the blocks: the pairs of the smallest exponential variates, whose
    rates are the pairs' weights."""
    sizes = torch.tensor(_block_sizes(n, blocks), device=DEV)
    label = torch.repeat_interleave(torch.arange(len(sizes), device=DEV), sizes)
    rate = torch.where(label[:, None] == label[None, :], 0.2 + 0.8 * len(sizes), 0.2)
    t = torch.empty((n, n), device=DEV).exponential_(generator=gen) / rate
    t[torch.ones((n, n), dtype=torch.bool, device=DEV).tril()] = math.inf
    m = min(int(n * degree / 2), n * (n - 1) // 2)
    key = torch.topk(t.flatten(), m, largest=False, sorted=False).indices
    return _csr_from_pairs(n, key // n, key % n)


def _graph(case, seed):
    gen = _gen(seed, 1)
    n = case["n"]
    kind = case.get("graph", "cl")
    if kind == "er":
        return _csr_from_pairs(n, *_uniform_pairs(n, case["degree"], gen))
    if kind == "sbm":
        return _sbm_dense(n, case["blocks"], case["p_in"], case["p_out"], gen)
    return _chung_lu(n, case["gamma"], case["degree"], gen)


def _csr(n, row_ptr, cols):
    return ops.Csr(n, int(cols.numel()), row_ptr, cols.to(torch.int32))


def _positions(k, gen, scale=1.0):
    return ((torch.rand((k, 2), device=DEV, generator=gen) * 2 - 1) * scale).contiguous()


def _sources(case, seed, row_ptr):
    n, k = case["n"], case["sources"]
    if k >= n:
        return torch.arange(n, dtype=torch.int32, device=DEV)
    live = torch.nonzero(torch.diff(row_ptr) > 0).flatten()
    pick = live[torch.randperm(live.numel(), device=DEV, generator=_gen(seed, 2))[:k]]
    return torch.sort(pick).values.to(torch.int32)


def _distances(k, seed):
    """PDist-like target distances: the distances of k points in a plane plus
    noise, brought into PDist's range [2, 2 ln k], symmetric, zero diagonal."""
    gen = _gen(seed, 3)
    p = torch.randn((k, 2), device=DEV, generator=gen)
    d = torch.cdist(p, p) + 0.3 * torch.rand((k, k), device=DEV, generator=gen)
    d = torch.triu(d, 1)
    hi = max(2.0 * math.log(k), 3.0)
    d = 2.0 + (hi - 2.0) * (d / d.max())
    d = torch.triu(d, 1)
    return (d + d.T).contiguous()


def _leaf_ranges(n, k):
    """k contiguous id ranges, the stand-in for the children of a supernode."""
    cut = torch.linspace(0, n, k + 1).round().to(torch.int32).to(DEV)
    return cut, torch.arange(n, dtype=torch.int32, device=DEV)


def _hub_leaves(n, k):
    """The k first nodes (the largest expected degrees) as singleton supernodes."""
    return torch.arange(k + 1, dtype=torch.int32, device=DEV), torch.arange(k, dtype=torch.int32, device=DEV)


def _batch_sizes(case):
    """Log-uniform sizes, evenly spread over their quantiles, shuffled."""
    g = case["graphs"]
    q = (np.arange(g) + 0.5) / g
    sizes = np.rint(np.exp(math.log(case["n_lo"]) + q * math.log(case["n_hi"] / case["n_lo"]))).astype(np.int64)
    return np.random.default_rng(7).permutation(sizes)


def _batch_blocks(i):
    return 4 + i * 5 % 13


def _batch_graphs(case, seed):
    """The disjoint union of the subgraphs: sizes, row_ptr, cols (host arrays)."""
    sizes = _batch_sizes(case)
    gen = _gen(seed, 4)
    ptrs, cols, node, arcs = [], [], 0, 0
    for i, n in enumerate(sizes.tolist()):
        rp, _, c = _sbm_dense(n, _batch_blocks(i), case["p_in"], case["p_out"], gen)
        ptrs.append(rp[:-1].to(torch.int64) + arcs)
        cols.append(c + node)
        node += n
        arcs += int(c.numel())
    ptrs.append(torch.tensor([arcs], device=DEV))
    return sizes, torch.cat(ptrs).to(torch.int32).cpu().numpy(), torch.cat(cols).to(torch.int32).cpu().numpy()


def prepare(case, seed):
    kind = case["kind"]
    if kind == "zoom":
        rp, _, cols = _graph(case, seed)
        return types.SimpleNamespace(case=case, g=_csr(case["n"], rp, cols), leaves=_hub_leaves(case["n"], case["k"]),
                                     x0=_positions(case["k"], _gen(seed, 5)))
    if kind == "level":
        rp, _, cols = _graph(case, seed)
        n, k = case["n"], case["k"]
        m, tau = int(cols.numel()), 1.0 / math.sqrt(k * n)
        # the paper's default threshold, eps = 1 - 1/e and delta = 1 / (10 k)
        r_max = (1 - 1 / math.e) / (10 * k) / (m * tau)
        return types.SimpleNamespace(case=case, g=_csr(n, rp, cols), leaves=_leaf_ranges(n, k), r_max=r_max)
    if kind == "ppr":
        rp, _, cols = _graph(case, seed)
        src = _sources(case, seed, rp)
        return types.SimpleNamespace(case=case, g=_csr(case["n"], rp, cols), src=src,
                                     tgt=None if case["sources"] >= case["n"] else src,
                                     x0=_positions(int(src.numel()), _gen(seed, 5)))
    if kind == "layout":
        return types.SimpleNamespace(case=case, delta=_distances(case["k"], seed),
                                     x0=_positions(case["k"], _gen(seed, 5), 4.0))
    if kind == "grad":
        rp, rows, cols, eid, ea, w, x = _training(case, seed)
        return types.SimpleNamespace(case=case, g=_csr(case["n"], rp, cols), arc_edge=eid, edge_arc=ea,
                                     w=w.requires_grad_(True), x=x.requires_grad_(True))
    sizes, rp, cols = _batch_graphs(case, seed)
    gb = types.SimpleNamespace(graphs=range(len(sizes)), sizes=sizes,
                               node_off=np.concatenate([[0], np.cumsum(sizes)]),
                               mat_off=np.concatenate([[0], np.cumsum(sizes * sizes)]), row_ptr=rp, col_idx=cols)
    b = ops.Batch(gb, DEV)
    bufs = b.buffers(_positions(b.n_nodes, _gen(seed, 5)))
    bufs["stress"] = None  # the optional stress output is not asked for
    return types.SimpleNamespace(case=case, bufs=bufs,
                                 plan=ops.BatchPlan(b, bufs, alpha=ALPHA, tol=case["tol"], stress_iters=case["sweeps"]))


def _training(case, seed):
    """Weighted block model: each undirected edge one weight near 1, from which
    training starts, and a spread-out layout."""
    n, gen = case["n"], _gen(seed, 1)
    rp, rows, cols = _sbm_edges(n, case["blocks"], case["degree"], gen)
    und = torch.minimum(rows, cols) * n + torch.maximum(rows, cols)
    _, eid = torch.unique(und, return_inverse=True)
    fwd = torch.nonzero(rows < cols).flatten()
    edge_arc = torch.empty(fwd.numel(), dtype=torch.int64, device=DEV)
    edge_arc[eid[fwd]] = fwd
    w = 0.75 + 0.5 * torch.rand(fwd.numel(), device=DEV, generator=gen)
    return rp, rows, cols, eid, edge_arc, w, _positions(n, gen, 4.0)


# --------------------------------------------------------------------- run

def run(state):
    case = state.case
    kind = case["kind"]
    if kind == "zoom":
        dppr, _, _, _ = ops.tau_push_level_dppr(state.g, state.leaves, alpha=ALPHA)
        delta = ops.pdist(dppr, case["n"])
        return {"dppr": dppr, "delta": delta, "x": ops.layout(delta, state.x0, case["sweeps"])}
    if kind == "level":
        return ops.gfp_level_dppr(state.g, state.leaves, alpha=ALPHA, r_max=state.r_max)[0]
    if kind == "ppr":
        ppr, dppr, pushes, _ = ops.ppr_matrix(state.g, state.src, tgt=state.tgt, alpha=ALPHA, tol=case["tol"])
        delta = ops.pdist(dppr, case["n"])
        out = {"ppr": ppr, "dppr": dppr, "delta": delta, "pushes": pushes}
        if case["sweeps"]:
            out["x"] = ops.layout(delta, state.x0, case["sweeps"])
        return out
    if kind == "layout":
        if case["exact"]:
            return ops.layout_step_exact(state.delta, state.x0, cg_tol=1e-6)[0]
        return ops.layout(state.delta, state.x0, case["sweeps"])
    if kind == "grad":
        state.w.grad = state.x.grad = None
        autograd.pprviz_loss(state.w, state.x, state.g, state.arc_edge, state.edge_arc, alpha=ALPHA,
                             T=case["T"]).backward()
        return {"w": state.w.grad, "x": state.x.grad}
    state.plan.launch()
    return {k: state.bufs[k] for k in ("x_out", "dppr", "delta")}


# -------------------------------------------------------------------- work

def _pushes(tol):
    return math.ceil(math.log(tol) / math.log(1 - ALPHA))


def _arcs(case):
    if case.get("graph") == "sbm":
        n, b = case["n"], min(case["blocks"], case["n"])
        return case["p_in"] * n * n / b + case["p_out"] * n * n * (1 - 1 / b)
    return case["n"] * case["degree"]


def work(case):
    """Each input read once, each output written once.  Operations: one add
    per arc, source and push (a multiply-add with weights), about 20 per pair
    and sweep of a layout."""
    kind = case["kind"]
    if kind == "zoom":
        # two sparse rounds at the least; everything small is read once
        arcs, k = _arcs(case), case["k"]
        return {"bytes": 4 * arcs + 8 * case["n"] + 12 * k * k, "flops": 2 * arcs * k + 20 * k * k * case["sweeps"]}
    if kind == "level":
        # every source's residue passes every arc at least once
        return {"bytes": 4 * _arcs(case) + 8 * case["n"], "flops": 2 * _arcs(case) * case["k"]}
    if kind == "ppr":
        n, s, m = case["n"], case["sources"], _arcs(case)
        return {"bytes": 4 * m + 4 * n + 12 * s * s,
                "flops": m * s * _pushes(case["tol"]) + 20 * s * s * (case["sweeps"] or 0)}
    if kind == "layout":
        k = case["k"]
        return {"bytes": 4 * k * k + 16 * k, "flops": 20 * k * k * case["sweeps"]}
    if kind == "grad":
        n, m = case["n"], case["n"] * case["degree"]
        return {"bytes": 16 * m + 16 * n, "flops": 2 * 2 * m * n * case["T"] + 2 * m * n + 40 * n * n}
    sizes = _batch_sizes(case).astype(float)
    blocks = np.array([4 + i * 5 % 13 for i in range(len(sizes))], dtype=float)
    arcs = case["p_in"] * sizes ** 2 / blocks + case["p_out"] * sizes ** 2 * (1 - 1 / blocks)
    return {"bytes": float(4 * arcs.sum() + 20 * sizes.sum() + 8 * (sizes ** 2).sum()),
            "flops": float((arcs * sizes).sum() * _pushes(case["tol"]) + 10 * (sizes ** 2).sum() * case["sweeps"])}


# ------------------------------------------------- the same in 64 bits

def _ppr64(n, row_ptr, rows, cols, src, T, w=None):
    """X[v, s] = pi_hat(src_s, v) after T pushes, FP64, and the degrees.  A node
    without arcs has a loop of its own."""
    w = torch.ones(cols.numel(), dtype=torch.float64, device=DEV) if w is None else w.double()
    d = torch.zeros(n, dtype=torch.float64, device=DEV).index_add_(0, rows, w)
    alone = torch.nonzero(torch.diff(row_ptr.long()) == 0).flatten()
    r, c = torch.cat([rows, alone]), torch.cat([cols, alone])
    v = torch.cat([w / d[cols], torch.ones(alone.numel(), dtype=torch.float64, device=DEV)])
    q = torch.sparse_coo_tensor(torch.stack([r, c]), (1 - ALPHA) * v, (n, n)).coalesce().to_sparse_csr()
    e = torch.zeros((n, src.numel()), dtype=torch.float64, device=DEV)
    e[src.long(), torch.arange(src.numel(), device=DEV)] = ALPHA
    x = e.clone()
    for _ in range(T - 1):
        x = torch.sparse.mm(q, x)
        x += e
    return x, d, q


def _pdist64(z, n):
    d = torch.clamp(torch.clamp(1.0 - torch.log(z), min=2.0), max=2.0 * math.log(n))
    d.fill_diagonal_(0.0)
    return d


def _sweeps64(delta, x, sweeps):
    delta, x = delta.double(), x.double()
    inv = torch.where(delta > 0, 1.0 / delta, 0.0)
    inv.fill_diagonal_(0.0)
    w = inv * inv
    sw = w.sum(1, keepdim=True)
    for _ in range(sweeps):
        dx, dy = x[:, None, 0] - x[None, :, 0], x[:, None, 1] - x[None, :, 1]
        c = inv / torch.sqrt(dx * dx + dy * dy + 1e-300)
        x = torch.where(sw > 0, (w @ x + torch.stack([(c * dx).sum(1), (c * dy).sum(1)], 1)) / sw, x)
    return x


def _exact_step64(delta, y):
    """The centred solution of L^w X = L^Y(Y) Y."""
    delta, y = delta.double(), y.double()
    k = y.shape[0]
    inv = torch.where(delta > 0, 1.0 / delta, 0.0)
    inv.fill_diagonal_(0.0)
    w = inv * inv
    diff = torch.sqrt((y[:, None, 0] - y[None, :, 0]) ** 2 + (y[:, None, 1] - y[None, :, 1]) ** 2)
    c = torch.where(diff > 0, inv / diff, 0.0)
    rhs = c.sum(1, keepdim=True) * y - c @ y
    lw = torch.diag(w.sum(1)) - w
    x = torch.linalg.solve(lw + 1.0 / k, rhs)  # adding the constant matrix fixes the centroid at zero
    return x - x.mean(0, keepdim=True)


def _grad64(case, seed):
    rp, rows, cols, eid, ea, w, x = _training(case, seed)
    n, T = case["n"], case["T"]
    wa, x = w.double()[eid], x.double()
    X, d, _ = _ppr64(n, rp, rows, cols, torch.arange(n, device=DEV), T, wa)
    pi = X.T.contiguous()
    z = d[:, None] * pi
    z = z + z.T
    raw = 1.0 - torch.log(z)
    hi = 2.0 * math.log(n)
    delta = _pdist64(z, n)
    eye = torch.eye(n, dtype=torch.bool, device=DEV)
    dx, dy = x[:, None, 0] - x[None, :, 0], x[:, None, 1] - x[None, :, 1]
    dist = torch.sqrt(dx * dx + dy * dy)
    safe = torch.where(eye, 1.0, delta)
    g = torch.where(eye, 0.0, 2.0 * (dist - delta) / (safe * safe) / torch.where(eye, 1.0, dist))
    gx = torch.stack([(g * dx).sum(1), (g * dy).sum(1)], 1)
    gd = torch.where(eye, 0.0, 2.0 * (1.0 - dist / safe) * dist / (safe * safe))
    G = torch.where(eye | ~((raw > 2.0) & (raw < hi)), 0.0, -gd / z)
    # adjoint: A = sum_{j<T} (Q^T)^j D G, Q = (1-alpha) D^-1 W
    qt = torch.sparse_coo_tensor(torch.stack([rows, cols]), (1 - ALPHA) * wa / d[cols], (n, n)).coalesce().to_sparse_csr()
    gb = d[:, None] * G
    A = gb.clone()
    for _ in range(T - 1):
        A = torch.sparse.mm(qt, A)
        A += gb
    dq = (A @ pi.T)[rows, cols]
    row = torch.zeros(n, dtype=torch.float64, device=DEV).index_add_(0, rows, wa / d[rows] * dq)
    arc = (1 - ALPHA) / d[rows] * (dq - row[rows]) + (G * pi).sum(1)[rows]
    gw = torch.zeros(w.numel(), dtype=torch.float64, device=DEV).index_add_(0, eid, arc)
    return {"w": gw, "x": gx}


def _batch64(case, seed):
    sizes, rp, cols = _batch_graphs(case, seed)
    rp, cols = torch.as_tensor(rp, device=DEV).long(), torch.as_tensor(cols, device=DEV).long()
    x0 = _positions(int(sizes.sum()), _gen(seed, 5))
    T = _pushes(case["tol"])
    out = {"x_out": [], "dppr": [], "delta": []}
    node = 0
    for n in sizes.tolist():
        a, b = int(rp[node]), int(rp[node + n])
        deg = torch.diff(rp[node:node + n + 1])
        rows = torch.repeat_interleave(torch.arange(n, device=DEV), deg)
        A = torch.zeros((n, n), dtype=torch.float64, device=DEV)
        A[rows, cols[a:b] - node] = 1.0
        A += torch.diag((deg == 0).double())
        q = (1 - ALPHA) * A / A.sum(0, keepdim=True)
        x = ALPHA * torch.eye(n, dtype=torch.float64, device=DEV)
        # X after T pushes = alpha sum_{t<T} q^t, by doubling
        s, p = torch.zeros_like(x), torch.eye(n, dtype=torch.float64, device=DEV)  # sum_{t<m} q^t, q^m, m = 0
        for bit in bin(T)[2:]:
            s, p = s + p @ s, p @ p
            if bit == "1":
                s, p = s + p, p @ q
        x = ALPHA * s
        dppr = deg.double()[:, None] * x.T
        delta = _pdist64(dppr + dppr.T, n)
        out["dppr"].append(dppr.flatten().cpu())
        out["delta"].append(delta.flatten().cpu())
        out["x_out"].append(_sweeps64(delta, x0[node:node + n], case["sweeps"]).cpu())
        node += n
    return {k: torch.cat(v) for k, v in out.items()}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("zoom", "level"):
        return None  # thresholded pushes: which of them are made is decided by rounding near the threshold
    if kind == "ppr":
        rp, rows, cols = _graph(case, seed)
        src = _sources(case, seed, rp)
        n, T = case["n"], _pushes(case["tol"])
        x, d, _ = _ppr64(n, rp, rows, cols, src, T)
        ppr = (x if case["sources"] >= n else x[src.long()]).T.contiguous()
        del x
        dppr = d[src.long()][:, None] * ppr
        delta = _pdist64(dppr + dppr.T, n)
        out = {"ppr": ppr, "dppr": dppr, "delta": delta, "pushes": None}
        if case["sweeps"]:
            out["x"] = (_sweeps64(delta, _positions(int(src.numel()), _gen(seed, 5)), case["sweeps"])
                        if src.numel() <= 4096 else None)
        return out
    if kind == "layout":
        delta, x0 = _distances(case["k"], seed), _positions(case["k"], _gen(seed, 5), 4.0)
        return _exact_step64(delta, x0) if case["exact"] else _sweeps64(delta, x0, case["sweeps"])
    if kind == "grad":
        return _grad64(case, seed)
    return _batch64(case, seed)
