"""GPU parity of the dense FP32 products on the matrix cores against FP64 torch
arithmetic, at the edges of their tiles and of the rules that choose them."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import ALPHA, get_ops

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

