"""GPU parity of the fidelity evaluation (eq. 7-8, Sec. 4.3; protocol of
Sec. 4.6) against the oracle: the two coalitions bit-exact for given phi
(ties, word boundaries, sparsity and top-k limits), the terms within the
coalition-value bar, the averages equal to the mean of the terms."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import fidelity as F
from oracle import gcn, sampler, subgraph
from paper_2401_04829_amd import _lib as L
from paper_2401_04829_amd.explainer import _vp
from tests.gpu_util import explainer_for, masks_np, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


def _gpu_masks(dev, phi, sparsity, top_k):
    M = len(phi)
    wpr = (M + 63) // 64
    p = torch.tensor(phi, dtype=torch.float32, device=dev)
    out = torch.full((2, wpr), -1, dtype=torch.int64, device=dev)
    L.gnnshap_fidelity_masks(_vp(p), M, sparsity, top_k, _vp(out), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return masks_np(out)


@pytest.mark.parametrize("M", [1, 2, 5, 63, 64, 65, 130, 1000, 1025, 5000])
def test_fidelity_masks_bit_exact(dev, M):
    """Random values, values with many ties (a few distinct magnitudes, both
    signs) and an all-equal vector; sparsities and top-k including 0, all
    and more than all."""
    rng = np.random.default_rng(M)
    cases = [rng.normal(size=M).astype(np.float32),
             (rng.integers(-3, 4, size=M) * 0.25).astype(np.float32),
             np.full(M, 0.5, dtype=np.float32)]
    for phi in cases:
        for s, k in [(0.3, 10), (0.0, 0), (1.0, M), (0.5, M + 3), (0.999, 1), (0.1, M // 2)]:
            got = _gpu_masks(dev, phi, s, k)
            keep, rest = F.fidelity_masks(phi, s, k)
            np.testing.assert_array_equal(got[0], sampler.pack(keep[None, :])[0], err_msg=f"G_S s={s}")
            np.testing.assert_array_equal(got[1], sampler.pack(rest[None, :])[0], err_msg=f"G_C-S k={k}")


def test_fidelity_terms_against_oracle(dev):
    """Cora-shaped targets explained on the GPU; their phi fed to both sides:
    the terms of eq. 7-8 within twice the coalition-value bar, the averages
    the mean of the terms, for the protocol of Sec. 4.6 and other settings."""
    cfg = W.make_config("cora")
    ex = explainer_for(cfg)
    targets = cfg["targets"][:8]
    exps = list(ex.explain_batch(targets, cfg["p"], cfg["seed"]))   # subgraphs stay valid together
    torch.cuda.synchronize()
    for sparsity, top_k in [(0.3, 10), (0.7, 3), (0.0, 0), (1.0, 10 ** 6)]:
        terms, avg = ex.fidelity(exps, sparsity, top_k)
        torch.cuda.synchronize()
        tg = terms.cpu().numpy().astype(np.float64)
        for t, (v, e) in enumerate(zip(targets, exps)):
            sub = subgraph.extract(cfg["indptr"], cfg["indices"], v, cfg["hops"])
            M = sub["num_edges"]
            game = gcn.Game(sub, cfg["X"], cfg["weights"], cfg["biases"])
            full_logits = game.logits(np.ones(M, bool))
            game.cls = gcn.predicted_class(full_logits)
            phi = e.phi.cpu().numpy()
            tm, tp, full = F.fidelity_terms(game, phi, sparsity, top_k)
            f_empty = game(np.zeros(M, bool))
            keep, rest = F.fidelity_masks(phi, sparsity, top_k)
            scale = max(abs(full), abs(f_empty), abs(game(keep)), abs(game(rest)))
            bar = 2e-4 * scale
            print("fidelity", v, sparsity, top_k, tg[t], (tm, tp, full), flush=True)
            assert abs(tg[t, 2] - full) <= 1e-4 * scale
            assert abs(tg[t, 0] - tm) <= bar, (v, tg[t, 0], tm)
            assert abs(tg[t, 1] - tp) <= bar, (v, tg[t, 1], tp)
        want = F.fidelity(tg)
        got = avg.cpu().numpy().astype(np.float64)
        assert abs(got[0] - want[0]) <= 1e-6 * max(1.0, abs(want[0]))
        assert abs(got[1] - want[1]) <= 1e-6 * max(1.0, abs(want[1]))


def test_fidelity_limits_exact(dev):
    """Removing every player leaves f(empty): with s = 1 and k >= M both terms
    are exactly |f(G_C) - f(empty)| as the device computes them (the empty
    coalition is pruned to f(empty), Sec. 3.4.1)."""
    cfg = W.make_config("tiny")
    ex = explainer_for(cfg)
    e = ex.explain(cfg["targets"][0], cfg["p"], cfg["seed"])
    terms, _ = ex.fidelity([e], 1.0, 10 ** 6)
    torch.cuda.synchronize()
    fef = e.f_empty_full.cpu().numpy().astype(np.float64)
    want = np.float32(abs(fef[1] - fef[0]))
    tg = terms.cpu().numpy()
    assert tg[0, 0] == want and tg[0, 1] == want
    assert tg[0, 2] == np.float32(fef[1])


@pytest.mark.parametrize("dims", [[12, 8, 3], [12, 33, 3], [12, 64, 3], [12, 8, 6, 3]])
def test_fidelity_batch_equals_single_calls(dev, dims):
    """gnnshap_fidelity_batch (one launch per step; three layers: target by
    target) against gnnshap_fidelity for targets of unlike sizes, bit for bit."""
    from paper_2401_04829_amd.explainer import Explainer
    indptr, indices = W.random_digraph(90, 400, seed=8, symmetric=True)
    Ws, bs = W.glorot_gcn(dims, 4, bias="random")
    ex = Explainer(indptr, indices, W.gaussian_features(90, 12, 5), Ws, bs, 2)
    targets = [int(v) for v in np.argsort(-np.diff(indptr))[[0, 3, 40, 80]]]
    exps = list(ex.explain_batch(targets, 400, 2))
    terms, _ = ex.fidelity(exps, 0.4, 5)
    one = torch.empty(3, device=dev)
    for t, e in enumerate(exps):
        ws = torch.empty(L.gnnshap_fidelity_workspace(e.sub.sg, ex.model), dtype=torch.uint8, device=dev)
        L.gnnshap_fidelity(e.sub.sg, ex.model, _vp(ex.X), -1, _vp(e.phi), 0.4, 5, _vp(one), _vp(ws), ws.numel(),
                           torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert torch.equal(one, terms[t]), (targets[t], one, terms[t])


def test_fidelity_captured_in_a_graph(dev):
    """Explainer.fidelity recorded in a graph and replayed on new phi, with
    eager calls on other targets between the replays (they use the host
    staging buffers again): every replay equals the eager result bit for bit."""
    cfg = W.make_config("cora")
    ex = explainer_for(cfg)
    exps = list(ex.explain_batch(cfg["targets"][:4], cfg["p"], cfg["seed"]))
    saved = [e.phi.clone() for e in exps]
    ex.fidelity(exps, 0.3, 4)                     # the workspace exists before the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        terms, avg = ex.fidelity(exps, 0.3, 4)
    for i in range(5):
        for e, p in zip(exps, saved):
            e.phi.copy_(torch.roll(p, i))
        for _ in range(3):
            want, want_avg = ex.fidelity(exps, 0.3, 4)
            ex.fidelity(exps[1:], 0.3, 4)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(terms, want) and torch.equal(avg, want_avg), i
