"""Coalition values of three-layer GCNs whose hidden widths the contraction on
matrix cores does not take: the products with the weight matrices on gathered
rows (no X W_1 prepared), on the boundary nodes' rows and on a number of rows
that the device counts, in the split form and in fp32."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import gcn, subgraph
from paper_2401_04829_amd import _lib as L
from paper_2401_04829_amd.explainer import Explainer, _vp
from tests.gpu_util import require_gpu, y_tolerance

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


def _setup(dims, seed):
    indptr, indices = W.random_digraph(160, 900, seed=seed, symmetric=True)
    X = W.gaussian_features(160, dims[0], seed + 1)
    Ws, bs = W.glorot_gcn(dims, seed + 2, bias="random")
    ex = Explainer(indptr, indices, X, Ws, bs, 2)
    v = int(np.argmax(np.diff(indptr)))
    sub = subgraph.extract(indptr, indices, v, 2)
    return ex, v, gcn.Game(sub, X, Ws, bs), sub["num_edges"], int(sub["dst_ptr"][1])


def _masks(M, k, indeg, seed):
    """Random coalitions, a quarter of them without an in-edge of the target (pruned)."""
    rng = np.random.default_rng(seed)
    sel = rng.random((k, M)) < rng.random((k, 1))
    sel[::4, :indeg] = False
    return sel


def _values(dev, ex, sub, sel):
    M = sub.num_edges
    wpr = (M + 63) // 64
    padded = np.zeros((sel.shape[0], wpr * 64), np.uint8)
    padded[:, :M] = sel
    words = torch.from_numpy(np.packbits(padded, axis=1, bitorder="little").view(np.int64).copy()).to(dev)
    k = sel.shape[0]
    y = torch.empty(k, device=dev)
    fef = torch.empty(2, device=dev)
    cls = torch.empty(1, dtype=torch.int32, device=dev)
    ws = torch.empty(L.gnnshap_eval_workspace(sub.sg, ex.model, k), dtype=torch.uint8, device=dev)
    L.gnnshap_eval_coalitions(sub.sg, ex.model, _vp(ex.X), -1, _vp(words), k, wpr, _vp(y), _vp(fef), _vp(cls), _vp(ws),
                              ws.numel(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return y, fef, int(cls.item())


@pytest.mark.parametrize("dims", [(140, 250, 100, 5), (140, 100, 50, 5), (30, 130, 70, 3)])
@pytest.mark.parametrize("prepared", [False, True])
def test_values_against_float64(dev, dims, prepared):
    print("dense values", dims, prepared, flush=True)
    ex, v, game, M, indeg = _setup(dims, 3)
    if prepared:
        ex.prepare()
    sub = ex.extract(v)
    sel = _masks(M, 230, indeg, 4)
    y, fef, cls = _values(dev, ex, sub, sel)
    full = game.logits(np.ones(M, bool))
    assert cls == int(np.argmax(full))
    game.cls = cls
    f0, f1 = game(np.zeros(M, bool)), float(full[cls])
    ref = game.values(sel)
    err = np.abs(y.cpu().numpy() - ref)
    assert (err <= y_tolerance(ref, f0, f1)).all(), err.max()
    assert np.all(np.abs(fef.cpu().numpy() - [f0, f1]) <= y_tolerance(np.array([f0, f1]), f0, f1))


@pytest.mark.parametrize("dims", [(140, 250, 100, 5), (30, 130, 70, 3)])
def test_values_do_not_depend_on_the_other_coalitions(dev, dims):
    """The same bits for a coalition evaluated again, among few others and in
    another order (the rows that are evaluated are listed by whichever
    wavefront comes first, so also the place in a pass changes from run to
    run)."""
    print("dense values, rows", dims, flush=True)
    ex, v, game, M, indeg = _setup(dims, 5)
    sub = ex.extract(v)
    sel = _masks(M, 6000, indeg, 6)
    y, fef, _ = _values(dev, ex, sub, sel)
    for _ in range(2):
        assert torch.equal(_values(dev, ex, sub, sel)[0], y)
    for rows in (np.arange(37), np.arange(5990, 6000), np.arange(6000)[::-1]):
        got = _values(dev, ex, sub, np.ascontiguousarray(sel[rows]))
        assert torch.equal(got[0], y[torch.from_numpy(rows.copy()).to(dev)])
        assert torch.equal(got[1], fef)
