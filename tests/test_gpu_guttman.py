"""GPU parity: the exact stress-majorization step (layout_step_exact, the
appendix's Guttman transform by conjugate gradients) through the C ABI,
against the FP64 oracle's pseudo-inverse step."""
import numpy as np
import pytest
import torch

import oracle as O
import synth
from gpu_util import get_ops

pytestmark = pytest.mark.gpu

CG_TOL = 1e-7
# Bar for one exact step, relative to the layout's scale.  L^w of a k-node
# layout is the Laplacian of the complete graph with weights Delta^-2, so its
# nonzero eigenvalues lie in [k w_min, k w_max] and its condition number on
# the centred subspace is at most (Delta_max / Delta_min)^2 <= (ln k)^2 for
# PDist values in [2, 2 ln k] (about 60 at k = 2304).  CG stopped at relative
# residual CG_TOL = 1e-7 in FP32 leaves a relative error of at most that
# condition number times (CG_TOL + a few u), below 1e-5 (the largest ratio
# measured on MI355X over these tests is 6.7e-7).
STEP_REL = 1e-5
WORST = [0.0]


def _step_close(err, scale, floor=0.0):
    ratio = (float(err) - floor) / float(scale)
    WORST[0] = max(WORST[0], ratio)
    print(f"[exact rel] {ratio:.3e} (worst so far {WORST[0]:.3e})", flush=True)
    assert ratio <= STEP_REL, ratio


@pytest.fixture(scope="module")
def ops():
    return get_ops()


def _t(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float32), device="cuda")


def _scale(a):
    return np.abs(a).max()


@pytest.mark.parametrize("k", [5, 97, 300, 1000])
def test_exact_step_matches_pseudo_inverse(ops, k):
    D = synth.random_distance_matrix(k, synth.BASE_SEED + k)
    Y = synth.uniform_layout(k, synth.BASE_SEED + k + 1)
    print(f"[guttman] k={k}", flush=True)
    x, iters = ops.layout_step_exact(_t(D), _t(Y), cg_tol=CG_TOL)
    want = O.majorization_step(Y.astype(np.float64), D.astype(np.float64))
    got = x.double().cpu().numpy()
    _step_close(np.abs(got - want).max(), _scale(want))
    assert 0 < iters < 1000
    np.testing.assert_allclose(got.mean(axis=0), 0.0, atol=1e-5 * _scale(want))


# Either side of the sizes up to which one block takes the whole solve (192) and
# the update and direction of an iteration (8192), by the residual that the step
# promises.
@pytest.mark.parametrize("k", [192, 193, 8192, 8193])
def test_exact_step_residual(ops, k):
    tol = 1e-4
    gen = torch.Generator(device="cuda").manual_seed(k)
    D = torch.rand((k, k), device="cuda", generator=gen) * 8 + 2
    D = torch.triu(D, 1)
    D = (D + D.T).contiguous()
    Y = (torch.rand((k, 2), device="cuda", generator=gen) * 2 - 1).contiguous()
    print(f"[guttman residual] k={k}", flush=True)
    x, iters = ops.layout_step_exact(D, Y, cg_tol=tol)
    assert 0 < iters < 100
    X, Y64 = x.double(), Y.double()
    b, r = torch.empty_like(Y64), torch.empty_like(Y64)
    for a in range(0, k, 1024):
        e = min(k, a + 1024)
        d = D[a:e].double()
        inv = torch.where(d > 0, 1.0 / d, 0.0)
        dist = (Y64[a:e, None] - Y64[None]).norm(dim=2)
        c = torch.where(dist > 0, inv / dist, 0.0)
        b[a:e] = c.sum(1, keepdim=True) * Y64[a:e] - c @ Y64
        r[a:e] = (inv * inv).sum(1, keepdim=True) * X[a:e] - (inv * inv) @ X - b[a:e]
    # The recursion stops at tol.  Its residual and the true one part by the FP32
    # row sums: 64 roundings of u = 2^-24 one after another at most (8192 columns
    # over 64 lanes and 4 waves, then the tree), times ||L^w|| ||x|| / ||b|| <= 4
    # (eigenvalues within a factor 4: the row sums of w are alike and its other
    # eigenvalues small), over at most 6 iterations: below tol again.
    assert (r.norm(dim=0) / b.norm(dim=0)).max().item() <= 2 * tol
    assert X.mean(0).abs().max().item() <= 1e-5 * X.abs().max().item()


def test_exact_steps_from_a_real_pdist_never_increase_stress(ops):
    # PDist of an ER graph (n = 500, mean degree 8) computed on the GPU, then
    # ten exact steps from a uniform start: the stress falls at every step.
    g = synth.erdos_renyi(500, 8, synth.BASE_SEED)
    csr = ops.Csr.from_graph(g, "cuda")
    _, dppr, _, _ = ops.ppr_matrix(csr, np.arange(g.n), tol=1e-6, want_ppr=False)
    delta = ops.pdist(dppr, g.n)
    D = delta.double().cpu().numpy()
    x = _t(synth.uniform_layout(g.n, synth.BASE_SEED + 1))
    s_prev = O.stress(x.double().cpu().numpy(), D)
    for step in range(10):
        X = x.double().cpu().numpy()
        x, iters = ops.layout_step_exact(delta, x, cg_tol=CG_TOL)
        got = x.double().cpu().numpy()
        want = O.majorization_step(X, D)
        _step_close(np.abs(got - want).max(), _scale(want))
        s = O.stress(got, D)
        assert s <= s_prev * (1 + 1e-6), (step, s, s_prev)
        s_prev = s


def test_planted_layout_is_a_fixed_point(ops):
    P, Dp = synth.planted_layout_distances(40, synth.BASE_SEED + 7)
    Pc = (P - P.mean(axis=0)).astype(np.float32)
    x, _ = ops.layout_step_exact(_t(Dp), _t(Pc), cg_tol=CG_TOL)
    _step_close(np.abs(x.double().cpu().numpy() - Pc).max(), _scale(Pc))


def test_coincident_points_and_converged_start(ops):
    # two coincident points: L^Y has no term for them, nothing is NaN
    k = 64
    D = synth.random_distance_matrix(k, synth.BASE_SEED + 50)
    Y = synth.uniform_layout(k, synth.BASE_SEED + 51)
    Y[7] = Y[3]
    x, _ = ops.layout_step_exact(_t(D), _t(Y), cg_tol=CG_TOL)
    got = x.double().cpu().numpy()
    assert np.all(np.isfinite(got))
    want = O.majorization_step(Y.astype(np.float64), D.astype(np.float64))
    _step_close(np.abs(got - want).max(), _scale(want))
    # a start that already solves its system stops before the first iteration
    x2, iters = ops.layout_step_exact(_t(D), x, cg_tol=1.0)
    assert iters == 0
    np.testing.assert_allclose(x2.double().cpu().numpy(), got - got.mean(axis=0), atol=1e-6 * _scale(got))


def test_iteration_cap_and_invalid_arguments(ops):
    from paper_2112_14944_amd import _lib
    k = 200
    D = _t(synth.random_distance_matrix(k, synth.BASE_SEED + 60))
    Y = _t(synth.uniform_layout(k, synth.BASE_SEED + 61))
    x, iters = ops.layout_step_exact(D, Y, cg_tol=0.0, cg_max_iter=3, allow_noconv=True)
    assert iters == 3 and torch.isfinite(x).all()
    for kwargs in (dict(cg_tol=-1.0), dict(cg_tol=float("nan")), dict(cg_max_iter=-1)):
        with pytest.raises(_lib.PprvizError) as ei:
            ops.layout_step_exact(D, Y, **kwargs)
        assert ei.value.status == _lib.PPR_EINVAL
    with pytest.raises(_lib.PprvizError) as ei:
        ops.layout_step_exact(D, Y, out=Y)
    assert ei.value.status == _lib.PPR_EINVAL


def test_4096_node_layout_solves_its_system(ops):
    # The size of the 4096-source layout of the 10^6-node graph: the defining
    # equation L^w X+ = L^Y(Y) Y checked in FP64 with the oracle's Laplacians.
    k = 4096
    D = synth.random_distance_matrix(k, synth.BASE_SEED + 70, hi=2.0 * np.log(1e6))
    Y = synth.uniform_layout(k, synth.BASE_SEED + 71)
    print("[guttman] k=4096", flush=True)
    x, iters = ops.layout_step_exact(_t(D), _t(Y), cg_tol=1e-6)
    X = x.double().cpu().numpy()
    D64 = D.astype(np.float64)
    rhs = O.laplacian_y(D64, Y.astype(np.float64)) @ Y.astype(np.float64)
    res = O.laplacian_w(D64) @ X - rhs
    assert np.linalg.norm(res[:, 0]) <= 2e-5 * np.linalg.norm(rhs[:, 0])
    assert np.linalg.norm(res[:, 1]) <= 2e-5 * np.linalg.norm(rhs[:, 1])
    np.testing.assert_allclose(X.mean(axis=0), 0.0, atol=1e-5 * _scale(X))


@pytest.mark.parametrize("k", [1, 2, 3])
def test_exact_step_tiny_layouts(ops, k):
    # k = 1: L^w = 0 and the centred solution is the origin; k = 2, 3: the
    # pseudo-inverse solution of a tiny system
    D = synth.random_distance_matrix(max(k, 2), synth.BASE_SEED + 80 + k)[:k, :k].copy()
    Y = synth.uniform_layout(k, synth.BASE_SEED + 90 + k)
    x, _ = ops.layout_step_exact(_t(D), _t(Y), cg_tol=CG_TOL)
    want = O.majorization_step(Y.astype(np.float64), D.astype(np.float64))
    got = x.double().cpu().numpy()
    _step_close(np.abs(got - want).max(), max(_scale(want), 1e-30), 1e-7)


# ------------------------------------------- batch form (one block per subgraph)


def _batch_case(ops, sizes, seed):
    """A batch of edgeless subgraphs of the given sizes (the exact step reads
    only node_off and mat_off), random distance matrices in the PDist pool
    and uniform random starts."""
    gb = synth.concat_graphs([synth.build_graph(int(n), [], []) for n in sizes])
    Ds = [synth.random_distance_matrix(max(int(n), 2), seed + i)[:n, :n].copy() for i, n in enumerate(sizes)]
    Ys = [synth.uniform_layout(int(n), seed + 500 + i) for i, n in enumerate(sizes)]
    batch = ops.Batch(gb)
    pool = _t(np.concatenate([D.ravel() for D in Ds]))
    x = _t(np.concatenate(Ys))
    return gb, batch, Ds, Ys, pool, x


def test_batch_exact_step_matches_pseudo_inverse(ops):
    # ragged sizes: 1 (the origin), 2, 3, a wave minus/plus one, several waves
    sizes = [1, 2, 3, 5, 63, 64, 65, 97, 300, 513]
    gb, batch, Ds, Ys, pool, x = _batch_case(ops, sizes, synth.BASE_SEED + 200)
    print(f"[guttman batch] sizes={sizes}", flush=True)
    out, iters, conv = ops.batch_step_exact(batch, pool, x, cg_tol=CG_TOL)
    got = out.double().cpu().numpy()
    iters = iters.cpu().numpy()
    assert np.all(conv.cpu().numpy() == 1)
    for g, n in enumerate(sizes):
        a, b = int(gb.node_off[g]), int(gb.node_off[g + 1])
        want = O.majorization_step(Ys[g].astype(np.float64), Ds[g].astype(np.float64))
        err = np.abs(got[a:b] - want).max()
        _step_close(err, max(_scale(want), 1e-30), 1e-7)
        assert 0 <= iters[g] < 1000


def test_batch_exact_step_at_the_largest_size_agrees_with_the_single_step(ops):
    # the largest subgraph (all five CG vectors in 92 KB of LDS) beside two
    # others; each subgraph against layout_step_exact on its own, and the
    # 2304-node one against its defining equation L^w X+ = L^Y(Y) Y in FP64
    sizes = [ops.batch_max_n(), 1000, 7]
    assert sizes[0] == 2304
    gb, batch, Ds, Ys, pool, x = _batch_case(ops, sizes, synth.BASE_SEED + 300)
    print(f"[guttman batch] sizes={sizes}", flush=True)
    out, iters, conv = ops.batch_step_exact(batch, pool, x, cg_tol=1e-6)
    got = out.double().cpu().numpy()
    assert np.all(conv.cpu().numpy() == 1)
    for g, n in enumerate(sizes):
        a, b = int(gb.node_off[g]), int(gb.node_off[g + 1])
        single, it1 = ops.layout_step_exact(_t(Ds[g]), _t(Ys[g]), cg_tol=1e-6)
        s = single.double().cpu().numpy()
        assert np.abs(got[a:b] - s).max() <= 1e-5 * _scale(s), n
        assert abs(int(iters[g]) - it1) <= 1, (n, int(iters[g]), it1)
    n = sizes[0]
    X = got[:n]
    D64 = Ds[0].astype(np.float64)
    Y64 = Ys[0].astype(np.float64)
    rhs = O.laplacian_y(D64, Y64) @ Y64
    res = O.laplacian_w(D64) @ X - rhs
    assert np.linalg.norm(res[:, 0]) <= 2e-5 * np.linalg.norm(rhs[:, 0])
    assert np.linalg.norm(res[:, 1]) <= 2e-5 * np.linalg.norm(rhs[:, 1])


def test_batch_exact_step_cap_and_invalid_arguments(ops):
    from paper_2112_14944_amd import _lib
    sizes = [40, 200]
    gb, batch, Ds, Ys, pool, x = _batch_case(ops, sizes, synth.BASE_SEED + 400)
    out, iters, conv = ops.batch_step_exact(batch, pool, x, cg_tol=0.0, cg_max_iter=2)
    assert np.all(iters.cpu().numpy() == 2) and np.all(conv.cpu().numpy() == 0)
    assert torch.isfinite(out).all()
    # two iterations from the same start match layout_step_exact's two
    for g in range(2):
        a, b = int(gb.node_off[g]), int(gb.node_off[g + 1])
        s, _ = ops.layout_step_exact(_t(Ds[g]), _t(Ys[g]), cg_tol=0.0, cg_max_iter=2, allow_noconv=True)
        sv = s.double().cpu().numpy()
        assert np.abs(out.double().cpu().numpy()[a:b] - sv).max() <= 1e-5 * _scale(sv)
    for kwargs in (dict(cg_tol=-1.0), dict(cg_tol=float("inf")), dict(cg_max_iter=-1)):
        with pytest.raises(_lib.PprvizError) as ei:
            ops.batch_step_exact(batch, pool, x, **kwargs)
        assert ei.value.status == _lib.PPR_EINVAL
    with pytest.raises(_lib.PprvizError) as ei:
        ops.batch_step_exact(batch, pool, x, out=x)
    assert ei.value.status == _lib.PPR_EINVAL


def test_batch_exact_step_on_the_batch_pipeline_output(ops):
    # 40 SBM subgraphs (sizes log-uniform in [32, 400]) through pprviz_batch
    # (all-pairs PPR, PDist, 20 Jacobi sweeps), then the exact step of every
    # subgraph from the sweeps' layout with the batch's own PDist pool: each
    # against the FP64 pseudo-inverse step on the same inputs, and the stress
    # of each subgraph does not rise (majorization)
    graphs = synth.sbm_batch(40, 32, 400, seed=synth.BASE_SEED + 600)
    gb = synth.concat_graphs(graphs)
    batch = ops.Batch(gb)
    x0 = torch.as_tensor(synth.uniform_layout(batch.n_nodes, synth.BASE_SEED + 601), device="cuda")
    bufs = ops.pprviz_batch(batch, batch.buffers(x0), stress_iters=20)
    print(f"[guttman batch] pipeline: {len(graphs)} subgraphs, {batch.n_nodes} nodes", flush=True)
    out, iters, conv = ops.batch_step_exact(batch, bufs["delta"], bufs["x_out"], cg_tol=CG_TOL)
    assert np.all(conv.cpu().numpy() == 1)
    xs = bufs["x_out"].double().cpu().numpy()
    got = out.double().cpu().numpy()
    for g in range(len(graphs)):
        a, b = int(gb.node_off[g]), int(gb.node_off[g + 1])
        D = ops.graph_block(gb, bufs["delta"], g).double().cpu().numpy()
        want = O.majorization_step(xs[a:b], D)
        _step_close(np.abs(got[a:b] - want).max(), _scale(want))
        assert O.stress(got[a:b], D) <= O.stress(xs[a:b], D) * (1 + 1e-6), g
