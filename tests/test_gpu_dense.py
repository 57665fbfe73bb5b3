"""GPU parity of the dense FP32 products on the matrix cores against FP64 torch
arithmetic, at the edges of their tiles and of the rules that choose them."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import ALPHA, get_ops, oracle_ppr

pytestmark = pytest.mark.gpu


def _walk64(g, device="cuda"):
    """W (FP64, dense), degrees, and Q = (1 - alpha) D^-1 W with the self-loop
    of a node without arcs."""
    n = g.n
    rows = torch.repeat_interleave(torch.arange(n), torch.as_tensor(np.diff(g.row_ptr)).long()).to(device)
    cols = torch.as_tensor(g.col_idx, device=device).long()
    w = torch.ones(g.nnz, dtype=torch.float64, device=device) if g.arc_weight is None else \
        torch.as_tensor(g.arc_weight, device=device).double()
    W = torch.zeros((n, n), dtype=torch.float64, device=device)
    W[rows, cols] = w
    d = W.sum(1)
    P = torch.where(d[:, None] > 0, W / torch.where(d > 0, d, 1.0)[:, None], torch.eye(n, device=device).double())
    return W, d, (1 - ALPHA) * P, rows, cols


# 63 .. 129: around the 64-wide tile; 300: several tiles, T = 2 takes the
# streaming adjoint and T = 40 the dense one; 3001: the 128-wide tile (from
# 3000 nodes on) with a ragged edge
@pytest.mark.parametrize("n,T", [(63, 40), (64, 40), (65, 40), (129, 40), (300, 2), (300, 40), (3001, 40)])
def test_weight_gradient_adjoint(n, T):
    ops = get_ops()
    nb = max(2, n // 100)
    g0 = synth.sbm(synth.equal_blocks(n, nb), min(1.0, 16.0 / (n / nb)), 4.0 / n, 40 + n, weighted=(0.5, 2.0, 41 + n))
    keep = (g0.eu != 5) & (g0.ev != 5)  # an isolated node
    g = synth.build_graph(n, g0.eu[keep], g0.ev[keep], g0.weight[keep])
    csr = ops.Csr.from_graph(g, "cuda")
    gen = torch.Generator(device="cuda").manual_seed(n)
    G = torch.randn((n, n), device="cuda", generator=gen)
    G = torch.triu(G, 1)
    G = (G + G.T).contiguous()
    print(f"[adjoint] n={n} nnz={g.nnz} T={T}", flush=True)
    got = ops.ppr_matrix_backward(csr, ALPHA, T, None, G).double()
    W, d, Q, rows, cols = _walk64(g)
    pi = torch.zeros_like(Q)
    A = torch.zeros_like(Q)
    Gb = d[:, None] * G.double()
    for _ in range(T):
        pi = ALPHA * torch.eye(n, dtype=torch.float64, device="cuda") + pi @ Q
        A = Gb + Q.T.contiguous() @ A
    dq = (A @ pi.T.contiguous())[rows, cols]
    wa = W[rows, cols]
    row = torch.zeros(n, dtype=torch.float64, device="cuda").index_add_(0, rows, wa / d[rows] * dq)
    arc = (1 - ALPHA) / d[rows] * (dq - row[rows]) + (G.double() * pi).sum(1)[rows]
    both = torch.zeros_like(Q)
    both[rows, cols] = arc
    want = (both + both.T)[rows, cols]
    # an entry of A is a sum of n FP32 terms in parts of 256 (at most
    # 256 + n / 256 roundings of u = 2^-24 one after another, 1.6e-5 of the
    # sum of the terms' sizes), everything after it FP64
    assert ((got - want).norm() / want.norm()).item() <= 2e-5


# Streaming adjoint steps (T = 3) on rows below and from 20 arcs on average, which
# gather a pass ahead or not: equal rows around the limit, and a few hubs.
@pytest.mark.parametrize("degree,hubs", [(6, 0), (18, 0), (20, 0), (40, 0), (6, 3)])
def test_weight_gradient_streaming_rows(degree, hubs):
    ops = get_ops()
    n, T = 2500, 3
    ring = np.concatenate([np.stack([np.arange(n), (np.arange(n) + k) % n], 1) for k in range(1, degree // 2 + 1)] +
                          [np.stack([np.full(n, h), np.arange(n)], 1) for h in range(hubs)])
    e = np.unique(np.sort(ring[ring[:, 0] != ring[:, 1]], 1), axis=0)
    g = synth.build_graph(n, e[:, 0], e[:, 1],
                          (0.5 + np.random.default_rng(degree).random(len(e))).astype(np.float32))
    csr = ops.Csr.from_graph(g, "cuda")
    G = torch.randn((n, n), device="cuda", generator=torch.Generator(device="cuda").manual_seed(n))
    G = (torch.triu(G, 1) + torch.triu(G, 1).T).contiguous()
    print(f"[streaming rows] nnz={g.nnz} degree={degree} hubs={hubs}", flush=True)
    # streamed, not dense
    assert (T - 1) * (4.0 * g.nnz * n / 11e12 + 6e-6) <= 2.0 * n**3 / 110e12 + 10e-6
    got = ops.ppr_matrix_backward(csr, ALPHA, T, None, G).double()
    W, d, Q, rows, cols = _walk64(g)
    pi = torch.zeros_like(Q)
    A = torch.zeros_like(Q)
    for _ in range(T):
        pi = ALPHA * torch.eye(n, dtype=torch.float64, device="cuda") + pi @ Q
        A = d[:, None] * G.double() + Q.T.contiguous() @ A
    dq = (A @ pi.T.contiguous())[rows, cols]
    row = torch.zeros(n, dtype=torch.float64, device="cuda").index_add_(0, rows, W[rows, cols] / d[rows] * dq)
    both = torch.zeros_like(Q)
    both[rows, cols] = (1 - ALPHA) / d[rows] * (dq - row[rows]) + (G.double() * pi).sum(1)[rows]
    want = (both + both.T)[rows, cols]
    # T steps of rows of at most n terms, summed by 8 arcs a pass: fewer roundings
    # than the dense products' 320, whose bar this is
    assert ((got - want).norm() / want.norm()).item() <= 2e-5


# One node past the graphs whose adjoint row is held in LDS, for a given pi: the
# dense adjoint pi^T D G / alpha and its product with pi at the arcs.
def test_weight_gradient_past_the_row_in_lds():
    ops = get_ops()
    n, T = 16385, 100
    g = synth.erdos_renyi(n, 18, 51)
    assert 2.0 * n**3 / 110e12 < (T - 1) * 4.0 * g.nnz * n / 11e12  # the dense adjoint
    csr = ops.Csr.from_graph(g, "cuda")
    pi = ops.ppr_matrix(csr, np.arange(n), alpha=ALPHA, tol=0.0, max_iter=T, want_dppr=False)[0]
    G = torch.randn((n, n), device="cuda", generator=torch.Generator(device="cuda").manual_seed(n))
    G = torch.triu(G, 1)
    G = (G + G.T).contiguous()
    print(f"[adjoint] n={n} nnz={g.nnz} T={T}", flush=True)
    got = ops.ppr_matrix_backward(csr, ALPHA, T, pi, G).double()
    rows = torch.repeat_interleave(torch.arange(n), torch.as_tensor(np.diff(g.row_ptr)).long()).cuda()
    cols = torch.as_tensor(g.col_idx, device="cuda").long()
    d = torch.as_tensor(np.diff(g.row_ptr), device="cuda").double()
    pi64 = pi.double()
    A = pi64.T.contiguous() @ (d[:, None] * G.double()) / ALPHA
    dq = torch.cat([(A[rows[e:e + 8192]] * pi64[cols[e:e + 8192]]).sum(1) for e in range(0, g.nnz, 8192)])
    row = torch.zeros(n, dtype=torch.float64, device="cuda").index_add_(0, rows, dq / d[rows])
    arc = (1 - ALPHA) / d[rows] * (dq - row[rows]) + (G.double() * pi64).sum(1)[rows]
    # the arc v -> u of u -> v: both lists are in row-major order
    rev = torch.argsort(cols * n + rows)
    want = arc + arc[rev]
    # as above: an entry of A is a sum of n FP32 terms, the rest FP64
    assert ((got - want).norm() / want.norm()).item() <= 2e-5


# rows of 1 to n - 1 arcs, so that a block's 32 arcs are many rows, one, or a
# part of one; 63, 64 and 513 around a wave's and eight waves' columns
@pytest.mark.parametrize("n", [63, 64, 257, 513, 1000])
def test_weight_gradient_hub_rows(n):
    ops = get_ops()
    T = 60
    rng = np.random.default_rng(n)
    eu = np.concatenate([np.zeros(n - 1, np.int64), np.arange(1, n - 1), rng.integers(n // 2, n - 1, 40 * (n // 16))])
    ev = np.concatenate([np.arange(1, n), np.arange(2, n), np.full(40 * (n // 16), n - 1)])
    e = np.unique(np.stack([eu, ev], 1), axis=0)
    g = synth.build_graph(n, e[:, 0], e[:, 1], (0.5 + rng.random(len(e))).astype(np.float32))
    csr = ops.Csr.from_graph(g, "cuda")
    G = torch.randn((n, n), device="cuda", generator=torch.Generator(device="cuda").manual_seed(n))
    G = (torch.triu(G, 1) + torch.triu(G, 1).T).contiguous()
    print(f"[hub rows] n={n} nnz={g.nnz}", flush=True)
    got = ops.ppr_matrix_backward(csr, ALPHA, T, None, G).double()
    W, d, Q, rows, cols = _walk64(g)
    pi = torch.zeros_like(Q)
    A = torch.zeros_like(Q)
    for _ in range(T):
        pi = ALPHA * torch.eye(n, dtype=torch.float64, device="cuda") + pi @ Q
        A = d[:, None] * G.double() + Q.T.contiguous() @ A
    dq = (A @ pi.T.contiguous())[rows, cols]
    row = torch.zeros(n, dtype=torch.float64, device="cuda").index_add_(0, rows, W[rows, cols] / d[rows] * dq)
    both = torch.zeros_like(Q)
    both[rows, cols] = (1 - ALPHA) / d[rows] * (dq - row[rows]) + (G.double() * pi).sum(1)[rows]
    want = (both + both.T)[rows, cols]
    # as above: an entry of A is a sum of n FP32 terms, the rest FP64
    assert ((got - want).norm() / want.norm()).item() <= 2e-5


def _series_plan(n, nnz, T):
    """The number of products and the pieces of the all-pairs series (the rule
    of csrc/ppr_dense.hpp)."""
    best, cost = (0, T, 0), 90 * T * nnz
    if n < 192 or n > 2304 or T < 24 or T > 4096:
        return best
    for k in (1, 2, 3):
        m = (T + k) // (k + 1)
        c = 100 * (m + 4) * nnz + 22 * k * n * (n + 64)
        if c < cost:
            cost, best = c, (k, m, T - k * m)
    return best


# sizes around the smallest graph that takes products (192), the change from
# 64- to 128-wide product tiles (512), the widths of the push tile (576, 1152)
# and the largest (2304); degrees and T that give every number of products,
# T = 24 and 25 the shortest series; and one that takes all pushes
@pytest.mark.parametrize("n,degree,T,k", [(191, 30, 86, 0), (192, 30, 86, 3), (193, 5, 86, 2), (511, 20, 86, 3),
                                          (512, 9, 86, 2), (513, 6, 86, 1), (577, 60, 24, 2), (640, 40, 25, 2),
                                          (1153, 50, 87, 3), (2304, 60, 86, 2), (2304, 8, 86, 0), (700, 40, 142, 3)])
def test_all_pairs_series(n, degree, T, k):
    ops = get_ops()
    g0 = synth.sbm(synth.equal_blocks(n, 4), min(1.0, 3.2 * degree / n), 0.27 * degree / n, 70 + n,
                   weighted=(0.5, 2.0, 71 + n))
    keep = (g0.eu != 9) & (g0.ev != 9)  # an isolated node
    g = synth.build_graph(n, g0.eu[keep], g0.ev[keep], g0.weight[keep])
    assert _series_plan(n, g.nnz, T)[0] == k, _series_plan(n, g.nnz, T)
    csr = ops.Csr.from_graph(g, "cuda")
    rng = np.random.default_rng(n)
    src = rng.permutation(n)
    tgt = rng.permutation(n)[: n // 2 + 1]
    print(f"[series] n={n} nnz={g.nnz} T={T} products={k}", flush=True)
    ppr, dppr, Tg, resid = ops.ppr_matrix(csr, src, tgt=tgt, tol=0.0, max_iter=T, check_residual=True)
    assert Tg == T
    _, d, Q, _, _ = _walk64(g)
    pi = torch.zeros_like(Q)
    for _ in range(T):
        pi = ALPHA * torch.eye(n, dtype=torch.float64, device="cuda") + pi @ Q
    s = torch.as_tensor(src, device="cuda").long()
    t = torch.as_tensor(tgt, device="cuda").long()
    want = pi[s][:, t]
    # the package's bars: PPR 1e-6, DPPR 1e-6 max(1, d(s)), residual 2e-6
    assert (ppr.double() - want).abs().max().item() <= 1e-6
    assert ((dppr.double() - d[s][:, None] * want) / d[s].clamp(min=1.0)[:, None]).abs().max().item() <= 1e-6
    assert np.abs(resid - (1.0 - pi[s].sum(1)).cpu().numpy()).max() <= 2e-6
    # the route without the series' buffers (the smaller workspace) agrees
    from paper_2112_14944_amd import _lib as L
    import ctypes as C
    cg = csr.c()
    lib = L.lib()
    small = torch.empty(lib.ppr_matrix_workspace(C.byref(cg), n, n), dtype=torch.uint8, device="cuda")
    assert lib.ppr_matrix_workspace_fast(C.byref(cg), n, n) >= small.numel() + (16 * n * n if n >= 192 else 0)
    out = torch.empty((n, n), device="cuda")
    si = s.to(torch.int32).contiguous()
    st = lib.ppr_matrix(C.byref(cg), C.c_void_p(si.data_ptr()), n, None, n, ALPHA, 0.0, T, C.c_void_p(out.data_ptr()),
                        None, None, None, C.c_void_p(small.data_ptr()), small.numel(),
                        C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == 0
    # either route rounds each value about T times by u = 2^-24, at random:
    # 1e-6 of the matrix's norm bounds the difference with room to spare
    assert ((out[:, t] - ppr).norm() / ppr.norm()).item() <= 1e-6


# Few sources: the iterate in HBM in slabs of 8, 16 and 32 columns (8 / 9 / 16 /
# 17 sources around their widths, 64 / 65 around a product tile), graphs of
# every size class, rows around and far above the 64 arcs of a whole-wave row
# (the power-law graphs), an isolated node among the sources, weights, T odd,
# even and short; targets that are the sources (about T / 2 pushes and one
# product), other targets, and all nodes.
@pytest.mark.parametrize("n,sources,T,targets", [
    (2000, 1, 86, "all"), (2000, 8, 85, "same"), (2300, 9, 86, "same"), (2305, 16, 87, "some"), (2305, 17, 8, "same"),
    (6000, 64, 86, "same"), (6000, 65, 99, "same"), (12000, 33, 7, "same"), (20000, 40, 100, "all"),
    (20000, 256, 60, "same"), (41000, 3, 86, "same"), (41000, 70, 31, "some"), (41000, 100, 41, "same")])
def test_few_sources(n, sources, T, targets):
    ops = get_ops()
    g0 = synth.chung_lu(n, 2.2, 20, 500 + n + sources)
    hub = int(np.argmax(np.diff(g0.row_ptr)))
    rng = np.random.default_rng(n + T)
    keep = (g0.eu != n - 2) & (g0.ev != n - 2)  # an isolated node
    w = (0.5 + 1.5 * rng.random(g0.m_und)).astype(np.float32) if T % 2 else None
    g = synth.build_graph(n, g0.eu[keep], g0.ev[keep], None if w is None else w[keep])
    src = rng.permutation(n)[:sources].astype(np.int32)
    src[0] = hub
    if sources > 2:
        src[1] = n - 2
    src = np.array(list(dict.fromkeys(src.tolist())), dtype=np.int32)  # distinct, unsorted
    csr = ops.Csr.from_graph(g, "cuda")
    sd = torch.as_tensor(src, device="cuda")
    tgt = {"all": None, "same": sd, "some": torch.as_tensor(rng.permutation(n)[:77].astype(np.int32), device="cuda")}
    tg = tgt[targets]
    print(f"[few] n={n} nnz={g.nnz} sources={len(src)} T={T} targets={targets}", flush=True)
    ppr, dppr, _, _ = ops.ppr_matrix(csr, sd, tgt=tg, tol=0.0, max_iter=T)
    ppr2, _, _, resid = ops.ppr_matrix(csr, sd, tgt=tg, tol=0.0, max_iter=T, check_residual=True)
    est, _, _, res, d = oracle_ppr(g, src, T=T)
    want = est if tg is None else est[:, tg.cpu().numpy()]
    # the package's bars: PPR 1e-6, DPPR 1e-6 max(1, d(s)), residual 2e-6
    for p in (ppr, ppr2):
        assert np.abs(p.double().cpu().numpy() - want).max() <= 1e-6
    dw = d[src][:, None] * want
    assert (np.abs(dppr.double().cpu().numpy() - dw) / np.maximum(1.0, d[src])[:, None]).max() <= 1e-6
    assert np.abs(resid - res).max() <= 2e-6


def _push64(g, src, T, alpha):
    """X[v, s] after T pushes in FP64, and the degrees; alpha as FP32 holds it."""
    rows = torch.repeat_interleave(torch.arange(g.n), torch.as_tensor(np.diff(g.row_ptr)).long()).cuda()
    cols = torch.as_tensor(g.col_idx, device="cuda").long()
    w = torch.ones(g.nnz, dtype=torch.float64, device="cuda") if g.arc_weight is None else \
        torch.as_tensor(g.arc_weight, device="cuda").double()
    d = torch.zeros(g.n, dtype=torch.float64, device="cuda").index_add_(0, rows, w)
    alone = torch.nonzero(d == 0).flatten()
    v = torch.cat([w / d[cols], torch.ones(alone.numel(), dtype=torch.float64, device="cuda")])
    a = float(np.float32(alpha))
    q = torch.sparse_coo_tensor(torch.stack([torch.cat([rows, alone]), torch.cat([cols, alone])]), (1 - a) * v,
                                (g.n, g.n)).coalesce().to_sparse_csr()
    e = torch.zeros((g.n, len(src)), dtype=torch.float64, device="cuda")
    e[torch.as_tensor(src, device="cuda").long(), torch.arange(len(src), device="cuda")] = a
    x = e.clone()
    for _ in range(T - 1):
        x = torch.sparse.mm(q, x)
        x += e
    return x, d


def _query(ops, csr, src, tgt, T, alpha, fast):
    """ppr_matrix with the fast or the general workspace: (ppr, dppr)."""
    import ctypes as C
    from paper_2112_14944_amd import _lib as L
    lib, cg = L.lib(), csr.c()
    k, m = src.numel(), csr.n if tgt is None else tgt.numel()
    size = lib.ppr_matrix_workspace_fast if fast else lib.ppr_matrix_workspace
    ws = torch.empty(size(C.byref(cg), k, m), dtype=torch.uint8, device="cuda")
    ppr, dppr = torch.empty((k, m), device="cuda"), torch.empty((k, m), device="cuda")
    p = lambda t: None if t is None else C.c_void_p(t.data_ptr())
    st = lib.ppr_matrix(C.byref(cg), p(src), k, p(tgt), m, alpha, 0.0, T, p(ppr), p(dppr), None, None, p(ws),
                        ws.numel(), C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == 0
    return ppr, dppr


# Many sources of a large graph, few pushes: the product that halves them holds
# half of the mass and sums over 200000 rows in few pieces.
def test_many_sources_short_series():
    ops = get_ops()
    n, k, T = 200000, 400, 8
    g = synth.chung_lu(n, 2.4, 24, 91)
    rng = np.random.default_rng(92)
    src = torch.as_tensor(np.sort(rng.choice(np.nonzero(np.diff(g.row_ptr))[0], k, replace=False)).astype(np.int32),
                          device="cuda")
    csr = ops.Csr.from_graph(g, "cuda")
    print(f"[short series] n={n} nnz={g.nnz} sources={k} T={T}", flush=True)
    half = _query(ops, csr, src, src, T, ALPHA, True)[0].double()
    full = _query(ops, csr, src, src[torch.arange(k)], T, ALPHA, False)[0].double()
    x, _ = _push64(g, src.cpu().numpy(), T, ALPHA)
    want = x[src.long()].T
    live = want > 0
    rel = lambda a, b: ((a - b)[live] / b[live]).pow(2).mean().sqrt().item()
    # One rounding of u = 2^-24 or so per push and value, and a row's sum of
    # positive terms: T u against FP64.  The two routes share the first half;
    # what is left are four pushes of one, and of the other a product whose FP32
    # sums have at most 128 terms (64 additions, sqrt(64 / 3) / 2 u of half the
    # mass) and a difference of two iterates: 6 u apart.
    assert not torch.equal(half, full)  # the halved route was taken
    assert rel(full, want) <= T * 2.0 ** -24
    assert rel(half, want) <= T * 2.0 ** -24
    assert rel(half, full) <= 6 * 2.0 ** -24


def _errors(got, want):
    """Norm of the error over the norm, and root mean square relative error of the entries."""
    got, live = got.double(), want != 0
    return ((got - want).norm() / want.norm()).item(), \
        ((got - want)[live] / want[live]).pow(2).mean().sqrt().item()


# Few sources take the iterate in HBM; the general workspace takes the LDS
# kernels.  The one route is no further from FP64 than the other: graphs with
# hubs (rows cut into parts there, taken by whole waves here), all targets, and
# the block among the sources by half the pushes.
@pytest.mark.parametrize("targets", ["all", "same"])
@pytest.mark.parametrize("n,gamma,weighted", [(2200, 2.3, False), (12000, 2.2, False), (12000, 2.6, True)])
def test_few_sources_precision(n, gamma, weighted, targets):
    ops = get_ops()
    k, T = 250 if n < 4000 else 120, 86  # few enough that the faster route is the iterate in HBM
    g0 = synth.chung_lu(n, gamma, 20, 700 + n)
    w = (0.5 + np.random.default_rng(7).random(g0.m_und)).astype(np.float32) if weighted else None
    g = synth.build_graph(n, g0.eu, g0.ev, w)
    live = np.nonzero(np.diff(g.row_ptr))[0]
    src = torch.as_tensor(np.sort(np.random.default_rng(8).choice(live, k, replace=False)).astype(np.int32),
                          device="cuda")
    csr = ops.Csr.from_graph(g, "cuda")
    tgt = src if targets == "same" else None
    print(f"[precision] n={n} nnz={g.nnz} sources={k} targets={targets}", flush=True)
    fast = _query(ops, csr, src, tgt, T, ALPHA, True)
    slow = _query(ops, csr, src, tgt, T, ALPHA, False)
    x, d = _push64(g, src.cpu().numpy(), T, ALPHA)
    want = (x if tgt is None else x[src.long()]).T
    # the largest entries, k of them, make the norm: their error is known to
    # about 1 / sqrt(2 k) of itself, 4.5% or 6.5%; three times that
    for f, s, v in ((fast[0], slow[0], want), (fast[1], slow[1], d[src.long()][:, None] * want)):
        ef, es = _errors(f, v), _errors(s, v)
        print("norm %.3g %.3g  entries %.3g %.3g" % (ef[0], es[0], ef[1], es[1]), flush=True)
        assert ef[0] <= 1.2 * es[0] and ef[1] <= 1.2 * es[1]


# All pairs by the series and by all pushes (the general workspace): the one is
# no further from FP64 than the other; every tile width, 1 to 3 products,
# weights, an isolated node.
@pytest.mark.parametrize("n,degree,T,k", [(300, 24, 86, 3), (500, 8, 86, 2), (513, 6, 86, 1), (1000, 24, 100, 2),
                                          (1000, 50, 86, 3), (1500, 40, 86, 2), (2304, 60, 86, 2)])
def test_all_pairs_precision(n, degree, T, k):
    ops = get_ops()
    g0 = synth.sbm(synth.equal_blocks(n, 4), min(1.0, 3.2 * degree / n), 0.27 * degree / n, 170 + n,
                   weighted=(0.5, 2.0, 171 + n))
    # every node on a ring as well: an isolated one holds all of its mass in one
    # entry, whose rounding alone would be the norm
    ring = np.stack([np.arange(n), (np.arange(n) + 1) % n])
    e = np.unique(np.sort(np.concatenate([np.stack([g0.eu, g0.ev]), ring], 1), axis=0), axis=1)
    w = (0.5 + 1.5 * np.random.default_rng(n).random(e.shape[1])).astype(np.float32)
    g = synth.build_graph(n, e[0], e[1], w if n % 500 else None)
    assert _series_plan(n, g.nnz, T)[0] == k, _series_plan(n, g.nnz, T)
    csr = ops.Csr.from_graph(g, "cuda")
    src = torch.as_tensor(np.random.default_rng(n).permutation(n).astype(np.int32), device="cuda")
    print(f"[precision] n={n} nnz={g.nnz} T={T} products={k}", flush=True)
    fast = _query(ops, csr, src, None, T, ALPHA, True)
    slow = _query(ops, csr, src, None, T, ALPHA, False)
    x, d = _push64(g, src.cpu().numpy(), T, ALPHA)
    # the n diagonal entries make most of the norm: their error is known to about
    # 1 / sqrt(2 n) of itself, 4.1% at n = 300; three times that
    for f, s, v in ((fast[0], slow[0], x.T), (fast[1], slow[1], d[src.long()][:, None] * x.T)):
        ef, es = _errors(f, v), _errors(s, v)
        print("norm %.3g %.3g  entries %.3g %.3g" % (ef[0], es[0], ef[1], es[1]), flush=True)
        assert ef[0] <= 1.12 * es[0] and ef[1] <= 1.12 * es[1]


# The routes that replace pushes by products, at other alphas.  Where they are
# taken (all pairs 0.1 to 0.4, few sources from 0.1 on) they are no further from
# FP64 than all pushes; elsewhere the faster workspace changes nothing.
@pytest.mark.parametrize("alpha,T", [(0.5, 40), (0.3, 50), (0.1, 132), (0.0999, 132), (0.05, 270), (0.01, 300)])
def test_other_alphas(alpha, T):
    ops = get_ops()
    g = synth.sbm(synth.equal_blocks(1000, 4), 0.1, 0.02, 61)
    csr = ops.Csr.from_graph(g, "cuda")
    src = torch.arange(g.n, dtype=torch.int32, device="cuda")
    assert _series_plan(g.n, g.nnz, T)[0] > 0
    h = synth.chung_lu(42000, 2.4, 20, 62)
    hsr = ops.Csr.from_graph(h, "cuda")
    live = np.nonzero(np.diff(h.row_ptr))[0]
    hs = torch.as_tensor(np.random.default_rng(63).choice(live, 250, replace=False).astype(np.int32), device="cuda")
    print(f"[alpha] {alpha} T={T}", flush=True)
    for c, gr, s, t in ((csr, g, src, None), (hsr, h, hs, hs)):
        fast, slow = _query(ops, c, s, t, T, alpha, True), _query(ops, c, s, t, T, alpha, False)
        if alpha < 0.1 or (alpha > 0.4 and t is None):
            assert torch.equal(fast[0], slow[0]) and torch.equal(fast[1], slow[1])
            continue
        x, d = _push64(gr, s.cpu().numpy(), T, alpha)
        want = (x if t is None else x[t.long()]).T
        # as in the tests at 0.15: the diagonal's 1000 and 250 entries make the norm,
        # three times 1 / sqrt(2 k)
        bar = 1 + 3 / (2 * s.numel()) ** 0.5
        for f, r, v in ((fast[0], slow[0], want), (fast[1], slow[1], d[s.long()][:, None] * want)):
            ef, es = _errors(f, v), _errors(r, v)
            print("norm %.3g %.3g  entries %.3g %.3g" % (ef[0], es[0], ef[1], es[1]), flush=True)
            assert ef[0] <= bar * es[0] and ef[1] <= bar * es[1]
    if not 0.1 <= alpha <= 0.4:
        gb = synth.concat_graphs([g])
        b = ops.Batch(gb, "cuda")
        bufs = ops.pprviz_batch(b, b.buffers(torch.zeros((g.n, 2), device="cuda")), alpha=alpha, tol=0.0, max_iter=T,
                                stress_iters=0)
        assert torch.equal(ops.graph_block(gb, bufs["dppr"], 0), _query(ops, csr, src, None, T, alpha, False)[1])


# Either side of the rule that halves a query's pushes: the product of k sources
# costs n k^2, the pushes it saves as much as their arcs and k.
@pytest.mark.parametrize("k,T,halved", [(120, 8, True), (250, 8, False), (400, 20, True), (600, 20, False)])
def test_few_sources_halved_where_faster(k, T, halved):
    ops = get_ops()
    n = 42000
    g = synth.chung_lu(n, 2.4, 8, 95)
    # 15 TFLOP/s against 9 TB/s of 4-byte values
    assert halved == (n * k / 15e12 < (T - 1 - T // 2) * g.nnz * 4 / 9e12)
    csr = ops.Csr.from_graph(g, "cuda")
    live = np.nonzero(np.diff(g.row_ptr))[0]
    src = torch.as_tensor(np.sort(np.random.default_rng(96).choice(live, k, replace=False)).astype(np.int32),
                          device="cuda")
    print(f"[halved] nnz={g.nnz} sources={k} T={T} {halved}", flush=True)
    fast, slow = _query(ops, csr, src, src, T, ALPHA, True)[0], _query(ops, csr, src, src, T, ALPHA, False)[0]
    assert torch.equal(fast, slow) != halved
    assert ((fast - slow).norm() / slow.norm()).item() <= 1e-6  # the routes' bar


# Either side of the rule between the LDS kernels and the iterate in HBM: a push of
# the iterate costs for its rows as well as for their arcs, and a few pushes of a
# small graph less than the product's launches.
@pytest.mark.parametrize("n,degree,k,T,among,hbm",
                         [(15000, 6, 256, 86, False, False), (15000, 6, 48, 86, False, True),
                          (300, 6, 1, 8, True, False), (20000, 6, 48, 86, True, True)])
def test_few_sources_route(n, degree, k, T, among, hbm):
    ops = get_ops()
    g = synth.erdos_renyi(n, degree, 97)
    csr = ops.Csr.from_graph(g, "cuda")
    live = np.nonzero(np.diff(g.row_ptr))[0]
    src = torch.as_tensor(np.sort(np.random.default_rng(98).choice(live, k, replace=False)).astype(np.int32),
                          device="cuda")
    tgt = src if among else None
    print(f"[route] n={n} nnz={g.nnz} sources={k} T={T} {hbm}", flush=True)
    fast, slow = _query(ops, csr, src, tgt, T, ALPHA, True)[0], _query(ops, csr, src, tgt, T, ALPHA, False)[0]
    assert torch.equal(fast, slow) != hbm
    assert ((fast - slow).norm() / slow.norm()).item() <= 1e-6  # the routes' bar
