"""GPU parity of the GAT variant (App. E) against the oracle's GAT game:
coalition values within the y bar (f(empty), f(E_c) and the explained class
exact), pruned coalitions equal to f(empty) exactly, Shapley values within
the phi bar, exhaustive sampling equal to the exact Shapley values of eq. 1."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import gat as G
from oracle import sampler, shapley, subgraph, wls
from paper_2401_04829_amd.explainer import GatExplainer
from tests.gpu_util import masks_np, require_gpu, y_tolerance

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


def _say(*a):
    print(*a, flush=True)


def _cora_gat():
    cfg = W.make_config("cora")
    P = W.glorot_gat(cfg["X"].shape[1], 8, 16, 7, 41, bias="random")   # 8 heads of 16 (App. E)
    return cfg, P


def _small(seed, heads, F, C, n=60, e=200):
    indptr, indices = W.random_digraph(n, e, seed=seed, symmetric=True)
    X = W.gaussian_features(n, 12, seed + 7)
    P = W.glorot_gat(12, heads, F, C, seed + 9, bias="random")
    return indptr, indices, X, P


def _check(ex, indptr, indices, X, P, v, p, seed, rows=None, target_class=-1):
    res = ex.explain(v, p, seed, target_class=target_class)
    torch.cuda.synchronize()
    sub = subgraph.extract(indptr, indices, v, 2)
    M = sub["num_edges"]
    game = G.GatGame(sub, X, P)
    full = game.logits(np.ones(M, bool))
    cls = int(np.argmax(full)) if target_class < 0 else target_class
    game.cls = cls
    f0, f1 = game(np.zeros(M, bool)), float(full[cls])
    assert int(res.cls.item()) == cls
    fef = res.f_empty_full.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(fef - [f0, f1]) <= y_tolerance(np.array([f0, f1]), f0, f1))
    pl = sampler.plan(M, p)
    m, w_ref = sampler.sample(pl, seed, v)
    np.testing.assert_array_equal(masks_np(res.masks), sampler.pack(m))
    k = m.shape[0]
    if rows is None:
        rows = np.arange(k)
    y_ref = game.values(m[rows])
    y = res.y.cpu().numpy().astype(np.float64)
    err = np.abs(y[rows] - y_ref)
    assert (err <= y_tolerance(y_ref, f0, f1)).all(), err.max()
    dead = ~m[:, : int(sub["dst_ptr"][1])].any(axis=1)
    assert np.all(res.y.cpu().numpy()[dead] == res.f_empty_full.cpu().numpy()[0])
    return res, game, m, w_ref, (f0, f1)


@pytest.mark.parametrize("heads,F,C", [(8, 16, 7), (1, 5, 3), (3, 20, 4), (4, 64, 2)])
def test_gat_values_small_graphs(dev, heads, F, C):
    """Every coalition of several targets of random graphs, widths across
    one to four features per lane."""
    indptr, indices, X, P = _small(heads * 100 + F, heads, F, C)
    ex = GatExplainer(indptr, indices, X, P)
    deg = np.diff(indptr)
    for v in np.argsort(-deg)[:3]:
        _say("gat small", heads, F, C, int(v))
        _check(ex, indptr, indices, X, P, int(v), 600, 3)


def test_gat_cora_values_and_phi(dev):
    """Cora-shaped targets, 8 heads of 16 (App. E): sampled coalition values
    within the y bar and phi within the phi bar of the oracle's least squares
    on the oracle's own values."""
    cfg, P = _cora_gat()
    ex = GatExplainer(cfg["indptr"], cfg["indices"], cfg["X"], P)
    for v in cfg["targets"][:3]:
        _say("gat cora", v)
        res, game, m, w, (f0, f1) = _check(ex, cfg["indptr"], cfg["indices"], cfg["X"], P, v, 2000, 7)
        assert int(res.info.item()) == 0
        phi_ref = wls.kernel_shap(m, w, game.values(m), f0, f1)
        phi = res.phi.cpu().numpy().astype(np.float64)
        assert np.abs(phi - phi_ref).max() <= 1e-3 * np.abs(phi_ref).max()


def test_gat_fixed_class(dev):
    cfg, P = _cora_gat()
    ex = GatExplainer(cfg["indptr"], cfg["indices"], cfg["X"], P)
    v = cfg["targets"][5]
    _check(ex, cfg["indptr"], cfg["indices"], cfg["X"], P, v, 1000, 2, rows=np.arange(0, 1000, 7), target_class=3)


def test_gat_exhaustive_equals_exact_shapley(dev):
    """A target with at most 10 players and every coalition sampled: the
    GPU explanation equals eq. 1 on the oracle's GAT game."""
    indptr, indices, X, P = _small(5, 8, 16, 4, n=80, e=120)
    deg = np.diff(indptr)
    ex = GatExplainer(indptr, indices, X, P)
    done = 0
    for v in np.argsort(-deg):
        sub = subgraph.extract(indptr, indices, int(v), 2)
        M = sub["num_edges"]
        if not 3 <= M <= 10:
            continue
        _say("gat exhaustive", int(v), M)
        res = ex.explain(int(v), 2 ** M - 2, 1)
        torch.cuda.synchronize()
        game = G.GatGame(sub, X, P)
        game.cls = int(np.argmax(game.logits(np.ones(M, bool))))
        assert int(res.cls.item()) == game.cls
        codes = np.arange(1 << M)
        table = np.array([game(((codes[i] >> np.arange(M)) & 1).astype(bool)) for i in range(1 << M)])
        exact = shapley.exact_shapley(table, M)
        phi = res.phi.cpu().numpy().astype(np.float64)
        assert np.abs(phi - exact).max() <= 1e-3 * np.abs(exact).max()
        done += 1
        if done == 2:
            break
    assert done > 0


def test_gat_batch_equals_single(dev):
    """gnnshap_gat_explain_batch (App. E through the batched entry points):
    for 12 Cora-shaped targets, with targets of a different fixed class as
    well, every output (masks, weights, coalition values, f(empty), f(E_c),
    class, phi, info) equals the single-target calls' bit for bit, and the
    batch's phi of the first target is within the phi bar of the oracle's
    least squares on the oracle's GAT values."""
    cfg, P = _cora_gat()
    ex = GatExplainer(cfg["indptr"], cfg["indices"], cfg["X"], P)
    targets = [int(v) for v in cfg["targets"][:12]]
    for target_class in (-1, 2):
        _say("gat batch", len(targets), "targets, class", target_class)
        batch = ex.explain_batch(targets, 2000, 7, target_class=target_class)
        torch.cuda.synchronize()
        for i, v in enumerate(targets):
            b = batch[i]
            s = ex.explain(v, 2000, 7, target_class=target_class)
            torch.cuda.synchronize()
            for name in ("masks", "weights", "y", "f_empty_full", "cls", "phi", "info"):
                assert torch.equal(getattr(b, name), getattr(s, name)), (v, target_class, name)
    b = ex.explain_batch(targets[:1], 2000, 7)[0]
    torch.cuda.synchronize()
    sub = subgraph.extract(cfg["indptr"], cfg["indices"], targets[0], 2)
    M = sub["num_edges"]
    game = G.GatGame(sub, cfg["X"], P)
    game.cls = int(np.argmax(game.logits(np.ones(M, bool))))
    assert int(b.cls.item()) == game.cls
    pl = sampler.plan(M, 2000)
    m, w = sampler.sample(pl, 7, targets[0])
    np.testing.assert_array_equal(masks_np(b.masks), sampler.pack(m))
    f0, f1 = game(np.zeros(M, bool)), game(np.ones(M, bool))
    phi_ref = wls.kernel_shap(m, w, game.values(m), f0, f1)
    phi = b.phi.cpu().numpy().astype(np.float64)
    assert np.abs(phi - phi_ref).max() <= 1e-3 * np.abs(phi_ref).max()


@pytest.mark.parametrize("heads,F", [(1, 16), (16, 16), (2, 48), (3, 20)])
def test_gat_lanes_and_batch_at_edges(dev, heads, F):
    """One coalition per lane (head widths that are multiples of 16) and per
    wavefront (20): 130 and 6 coalitions (a part of a workgroup), 1 to 256
    features, a hub with more than 64 in-neighbours, a target with a single
    one; the batch (targets of unlike sizes in one launch) equals the single
    calls bit for bit."""
    rng = np.random.default_rng(heads * 100 + F)
    hub = np.stack([np.arange(1, 81), np.zeros(80, np.int64)])
    rest = rng.integers(1, 90, size=(2, 60))
    e = np.concatenate([hub, rest, [[85], [95]], [[95], [96]]], axis=1)   # 96 <- 95 <- 85
    indptr, indices = W.in_csr_from_directed(97, e[0], e[1])
    X = W.gaussian_features(97, 9, 3)
    P = W.glorot_gat(9, heads, F, 5, 11, bias="random")
    ex = GatExplainer(indptr, indices, X, P)
    targets = [0, 96]
    for p in (130, 6):
        single = [_check(ex, indptr, indices, X, P, v, p, 3)[0] for v in targets]
        single = [(r.y.clone(), r.f_empty_full.clone(), r.cls.clone()) for r in single]
        batch = ex.explain_batch(targets, p, 3)
        torch.cuda.synchronize()
        for t in range(len(targets)):
            for a, b in zip(single[t], (batch[t].y, batch[t].f_empty_full, batch[t].cls)):
                assert torch.equal(a, b)


def _star(dev, n, X, P):
    """Node 0 with the in-neighbours 1 .. n, which have none."""
    indptr, indices = W.in_csr_from_directed(n + 1, np.arange(1, n + 1), np.zeros(n, np.int64))
    return GatExplainer(indptr, indices, X, P), indptr, indices


@pytest.mark.parametrize("heads,F", [(16, 16), (8, 16), (4, 64), (3, 80), (4, 20)])
def test_gat_sums_over_features_are_pairwise(dev, heads, F):
    """The layer-2 sums of one feature of 1 and many just below half its last
    place: added one after the other to the 1 they are lost (15 of 16, or all
    of them), added in pairs they count.  All nodes have the same layer-1 row
    (W_1 = 0) and the same logits, so a target with one in-neighbour has
    exactly that sum as its value.  Bound: half a unit in the last place of
    the sum (2^-23 of it at most) per level of a tree over 256 features, and
    one for the division."""
    nf, s = heads * F, 0.99 * 2.0 ** -24
    b1 = np.full(nf, s, np.float32)
    P = dict(W1=np.zeros((3, nf), np.float32), att_src1=np.zeros((heads, F), np.float32),
             att_dst1=np.zeros((heads, F), np.float32), b1=b1, W2=np.ones((nf, 2), np.float32),
             att_src2=np.zeros(2, np.float32), att_dst2=np.zeros(2, np.float32), b2=np.zeros(2, np.float32))
    for at in (0, nf // 2 + 3, nf - 1):
        _say("gat sums", heads, F, at)
        P["b1"] = b1.copy()
        P["b1"][at] = 1.0
        ex, indptr, indices = _star(dev, 2, np.ones((3, 3), np.float32), P)
        res = ex.explain(0, 2, 1)
        torch.cuda.synchronize()
        exact = 1.0 + (nf - 1) * float(np.float32(s))
        got = np.concatenate([res.y.cpu().numpy(), res.f_empty_full.cpu().numpy()]).astype(np.float64)
        assert np.abs(got - exact).max() <= 9 * 2.0 ** -24 * exact, (got - exact) * 2.0 ** 24


@pytest.mark.parametrize("F", [16, 20])
@pytest.mark.parametrize("plus,minus", [((1,), ()), ((6,), ()), ((17,), ()), ((17,), (1, 6, 22)), ((), (6,)),
                                        ((), (6, 22)), ((), (1,)), ((3, 6), ()), ((6, 22), ())])
def test_gat_infinite_logits(dev, F, plus, minus):
    """In-neighbours whose layer-2 logit overflows to +inf or -inf (finite
    features): f(E_c) and the coalition values follow one rule wherever the
    neighbour stands: one +inf takes all the weight, two leave no number, -inf
    has none.  The finite logits are so far apart that the largest one (equal
    for all other neighbours) takes the rest."""
    _say("gat infinite logits", F, plus, minus)
    n = 24
    X = np.zeros((n + 1, 3), np.float32)
    X[:, 0], X[:, 1] = 0.5, 1.0
    X[0, 0] = 0.1
    X[list(plus), 0] = 2.0
    X[list(minus), 2] = 2.0
    W1 = np.zeros((3, F), np.float32)
    W1[0, 0], W1[1, 1], W1[2, 2] = 1.0, 0.3, 1.0
    W2 = np.zeros((F, 2), np.float32)
    W2[:, 0] = 0.25
    W2[0, 1], W2[2, 1] = 1.0, -1.0
    P = dict(W1=W1, att_src1=np.zeros((1, F), np.float32), att_dst1=np.zeros((1, F), np.float32),
             b1=np.zeros(F, np.float32), W2=W2, att_src2=np.array([0.0, 3e38], np.float32),
             att_dst2=np.zeros(2, np.float32), b2=np.zeros(2, np.float32))
    ex, indptr, indices = _star(dev, n, X, P)
    res = ex.explain(0, 200, 1, target_class=0)
    torch.cuda.synchronize()
    rows = 0.25 * (X[:, 0] + 0.3 + X[:, 2])          # a node's layer-1 row times W_2[:, 0], ELU the identity

    def value(has):
        many = [j for j in plus if has[j - 1]]
        rest = [j for j in range(1, n + 1) if has[j - 1] and j not in plus and j not in minus]
        if many:
            return rows[many[0]] if len(many) == 1 else np.nan
        if rest:
            return rows[rest[0]]
        return None                                   # v alone beside neighbours of no weight

    sel = sampler.unpack(masks_np(res.masks), n)
    want = [value(s) for s in sel]
    keep = [i for i, w in enumerate(want) if w is not None]
    assert len(keep) > 100
    np.testing.assert_allclose(res.y.cpu().numpy()[keep], [want[i] for i in keep], rtol=1e-6)
    np.testing.assert_allclose(res.f_empty_full.cpu().numpy()[1], value(np.ones(n, bool)), rtol=1e-6)
