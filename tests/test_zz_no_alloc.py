"""ppr_matrix_noalloc, the entry point that allocates nothing, against
ppr_matrix on the same inputs: two calls in a row on one GPU (the second on
a smaller graph, so that it runs over the first call's leftovers in the
shared scratch array), each compared bit for bit, since both entry points
run the same kernels in the same order; plus the size limit."""
import ctypes as C

import numpy as np
import pytest
import torch

import synth
from gpu_util import ALPHA, get_ops

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ops():
    return get_ops()


def _both(ops, g, src, tgt, weighted):
    csr = ops.Csr.from_graph(g, "cuda", weighted=weighted)
    ppr, dppr, T, resid = ops.ppr_matrix(csr, src, tgt=tgt, alpha=ALPHA, tol=1e-6, check_residual=True)
    n_tgt = g.n if tgt is None else len(tgt)
    ppr2 = torch.full((len(src), n_tgt), float("nan"), device="cuda")
    dppr2 = torch.full_like(ppr2, float("nan"))
    T2, resid2 = ops.ppr_matrix_noalloc(csr, src, tgt=tgt, alpha=ALPHA, tol=1e-6, ppr=ppr2, dppr=dppr2,
                                        check_residual=True)
    torch.cuda.synchronize()
    assert T2 == T == 86
    assert torch.equal(ppr2, ppr) and torch.equal(dppr2, dppr)
    np.testing.assert_array_equal(resid2, resid)
    return ppr2


def test_noalloc_matches_ppr_matrix_two_calls(ops):
    # first call: weighted SBM, 1500 nodes (16-column tiles), all sources
    g1 = synth.sbm(synth.equal_blocks(1500, 6), 0.08, 0.004, 41, weighted=(0.5, 2.0, 42))
    print(f"[noalloc] call 1: n={g1.n} nnz={g1.nnz} weighted, all sources", flush=True)
    _both(ops, g1, np.arange(g1.n), None, True)
    # second call, smaller: unweighted ER, 300 nodes (64-column tiles), 70
    # sources and 90 targets
    g2 = synth.erdos_renyi(300, 8, 43)
    src = synth.random_sources(g2, 70, 44)
    tgt = np.sort(np.random.default_rng(45).choice(g2.n, 90, replace=False)).astype(np.int32)
    print(f"[noalloc] call 2: n={g2.n} nnz={g2.nnz}, {len(src)} sources x {len(tgt)} targets", flush=True)
    _both(ops, g2, src, tgt, False)


def test_noalloc_rejects_oversized_workspace(ops):
    from paper_2112_14944_amd import _lib as L
    g = synth.erdos_renyi(6000, 20, 46)  # mid-size path: its workspace exceeds the scratch array
    csr = ops.Csr.from_graph(g, "cuda")
    cg = csr.c()
    assert L.lib().ppr_matrix_workspace(C.byref(cg), g.n, g.n) > L.lib().ppr_matrix_noalloc_max_scratch()
    with pytest.raises(L.PprvizError) as ei:
        ops.ppr_matrix_noalloc(csr, np.arange(g.n), ppr=torch.empty((g.n, g.n), device="cuda"))
    assert ei.value.status == L.PPR_EUNSUPPORTED


# Run in a process of its own: the first uses of the library there.
_FIRST_USE = """
import numpy as np, torch, synth
from gpu_util import get_ops
ops = get_ops()
g = synth.erdos_renyi(300, 8, 1)
csr = ops.Csr.from_graph(g, "cuda")
src = torch.arange(g.n, dtype=torch.int32, device="cuda")
out = torch.zeros((g.n, g.n), device="cuda")
spare = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
del spare  # stays with the allocator for the calls below
torch.cuda.synchronize()
free = lambda: torch.cuda.mem_get_info()[0]
before = free()
want = ops.ppr_matrix(csr, src)[0]
torch.cuda.synchronize()
held = before - free()
s = torch.cuda.Stream()
graph = torch.cuda.CUDAGraph()
with torch.cuda.graph(graph, stream=s):  # the first call that needs the array is a captured one
    ops.ppr_matrix_noalloc(csr, src, ppr=out)
for _ in range(3):
    out.zero_()
    graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(out, want)
print("HELD", held)
"""


def test_noalloc_array_is_held_by_its_callers_only():
    # The array (93 MB) comes with the first call that uses it, which may be a
    # captured one; code alone is a few MB.
    import os
    import subprocess
    import sys
    here = os.path.dirname(os.path.abspath(__file__))
    env = dict(os.environ, PYTHONPATH=os.pathsep.join([os.path.dirname(here), here]))
    r = subprocess.run([sys.executable, "-c", _FIRST_USE], capture_output=True, text=True, timeout=100, env=env)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    words = r.stdout.split()
    held = int(words[words.index("HELD") + 1])
    print(f"[memory] ppr_matrix holds {held / 1e6:.1f} MB", flush=True)
    assert held < 50e6


# The iterates of 250 sources of 32000 and 39000 nodes, 65 and 80 MB, fit the
# array's room for the faster routes' buffers, the product's pieces do not as well;
# of 3000 nodes all of them fit.
@pytest.mark.parametrize("n,arcs,k", [(32000, 2000, 250), (39000, 2000, 250), (3000, 40000, 64)])
def test_noalloc_query_among_its_sources(ops, n, arcs, k):
    from paper_2112_14944_amd import _lib as L
    rng = np.random.default_rng(n)
    g = synth.build_graph(n, rng.integers(0, n, arcs // 2), rng.integers(0, n, arcs // 2))
    csr = ops.Csr.from_graph(g, "cuda")
    src = torch.as_tensor(np.sort(rng.choice(n, k, replace=False)).astype(np.int32), device="cuda")
    cg = csr.c()
    assert L.lib().ppr_matrix_workspace(C.byref(cg), k, k) <= L.lib().ppr_matrix_noalloc_max_scratch()
    print(f"[noalloc] n={n} nnz={g.nnz} {k} sources", flush=True)
    want = ops.ppr_matrix(csr, src, tgt=src)[1].double()
    got = torch.full((k, k), float("nan"), device="cuda")
    ops.ppr_matrix_noalloc(csr, src, tgt=src, dppr=got)
    # the same T pushes, halved or not: each value rounded about T = 86 times by
    # 2^-24 at random
    assert ((got.double() - want).norm() / want.norm()).item() <= 1e-6
