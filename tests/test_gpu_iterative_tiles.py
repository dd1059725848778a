"""The iterative solver's products on the matrix cores at the edges of their
tiles: players and bit rows around 16, 32, 64 and the 64- and 96-wide
workgroups, with and without sparse rows, and more rows than one fp32
accumulation segment holds."""
import numpy as np
import pytest
import torch

from oracle import sampler
from paper_2401_04829_amd import _lib as L
from paper_2401_04829_amd.explainer import _vp
from tests.gpu_util import masks_np, require_gpu, sample_on_gpu
from tests.test_gpu_iterative import _game, _oracle_rows, _solve

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


@pytest.mark.parametrize("M,p", [(2, 2), (15, 400), (16, 130), (17, 4000), (63, 1000), (64, 1026), (65, 1100),
                                 (95, 1500), (97, 1600), (128, 3000), (129, 2050), (257, 5000), (769, 4200),
                                 (1537, 9000)])
def test_products_at_tile_edges(dev, M, p):
    """phi against the exact solution of the projected normal equations on
    the oracle's rows.  Bound: the iteration stops at |A psi - b| <= 1e-6 |b|,
    so |psi - psi*|_2 <= 1e-6 |b| / lambda_min (A on 1-perp), plus the fp32
    rounding of phi and of f(full) - f(empty)."""
    print("iterative tiles", M, p, flush=True)
    plan, classes, masks, _ = sample_on_gpu(M, p, 5, 6)
    plan.iterative_threshold = 1
    mb, w = _oracle_rows(plan, masks, 5, 6)
    v, f0, f1 = _game(M, mb, 3 * M)
    yv = v(mb).astype(np.float32)
    fef = np.array([f0, f1], np.float32)
    phi, info = _solve(dev, plan, classes, masks, torch.tensor(yv, device=dev), torch.tensor(fef, device=dev))
    delta = float(fef[1]) - float(fef[0])
    P = mb - mb.mean(1, keepdims=True)
    A = (P * w[:, None]).T @ P
    b = P.T @ (w * (yv.astype(np.float64) - float(fef[0]) - delta / M * mb.sum(1)))
    lam = np.linalg.eigvalsh(A + A.trace() / M * np.full((M, M), 1.0 / M))[0]
    if info != 0:      # fewer random rows than unknowns: reported, as documented
        assert info == M + 1 and plan.random_begin == 0 and plan.num_rows // 2 < M - 1
        return
    ref = delta / M + np.linalg.lstsq(A + A.trace() / M * np.full((M, M), 1.0 / M), b, rcond=None)[0]
    bound = 1e-6 * np.linalg.norm(b) / lam + 1e-6 * np.linalg.norm(ref)
    assert np.linalg.norm(phi - ref) <= bound, (np.linalg.norm(phi - ref), bound)


def _linear_and_tanh(masks, M, a):
    at = torch.arange(64, device=masks.device)
    out = []
    for m in masks.split(1 << 14 if M > 64 else 1 << 20):
        t = ((m[:, :, None] >> at) & 1).view(m.shape[0], -1)[:, :M].float() @ a
        out.append(t + torch.tanh(t))
    return torch.cat(out)


def _factored_and_iterative(dev, M, p):
    """phi of the same rows by the factored solver (exact counts) and iteratively."""
    plan, classes, masks, _ = sample_on_gpu(M, p, 7, 8)
    g = torch.Generator(device=dev)
    g.manual_seed(9)
    a = torch.randn(M, generator=g, device=dev) / M ** 0.5
    y = _linear_and_tanh(masks, M, a)
    fef = torch.stack([torch.zeros((), device=dev), a.sum() + torch.tanh(a.sum())])
    got = []
    for threshold in (1 << 30, 1):
        plan.iterative_threshold = threshold
        phi, info = _solve(dev, plan, classes, masks, y, fef)
        assert info == 0
        got.append(phi)
    return plan, got


@pytest.mark.parametrize("M,p", [(8200, 2_300_000), (64, 18_400_000)])
def test_more_rows_than_one_accumulation_segment(dev, M, p):
    """More bit rows than the 512 x 8 groups of 256 (1,048,576) whose digit
    sums fp32 is sure to hold: more than 128 word columns, where a workgroup
    of pass B takes all of them and empties its sums between segments (lost or
    doubled ones would show; that a segment's sum is exact is asserted where
    its length is defined), and few columns, where they are taken in parts.
    Against the factored solver on the same rows, within the iteration's 1e-6
    and the factorisation's fp32."""
    print("iterative segments", M, p, flush=True)
    plan, (want, got) = _factored_and_iterative(dev, M, p)
    sparse = 64 * 1024 if M >= 128 else 0            # at most: kept as lists
    assert plan.num_rows // 2 - plan.random_begin - sparse > 512 * 8 * 256
    assert np.abs(got - want).max() <= 1e-4 * np.abs(want).max()


@pytest.mark.parametrize("M,p", [(64, 397_000), (64, 397_500), (65, 400_000), (127, 500_002), (200, 700_000),
                                 (2000, 560_000)])
def test_bit_rows_in_parts(dev, M, p):
    """Pass B's products whole just below 3,072 blocks of 64 bit rows and in
    parts from there on (of equal and unequal length, the last one shorter),
    one to 32 word columns.  Against the factored solver on the same rows."""
    print("iterative parts", M, p, flush=True)
    plan, (want, got) = _factored_and_iterative(dev, M, p)
    assert np.abs(got - want).max() <= 1e-4 * np.abs(want).max()


@pytest.mark.parametrize("order", ["as planned", "small sizes mixed", "descending"])
def test_class_tables_in_any_order(dev, order):
    """The random classes of a plan in another order of sizes, as the solve
    accepts them (the sparse rows are the first ones of small sizes): phi
    against the exact solution of the projected normal equations on these
    rows; bound as for the tile edges."""
    M, p = 1300, 30000
    print("class order", order, flush=True)
    plan, classes = L.gnnshap_plan_samples(M, p, 3, 4)
    plan.iterative_threshold = 1
    full = [c for c in classes if c.full]
    rand = [c for c in classes if not c.full]
    if order == "small sizes mixed":
        few = [c for c in rand if c.size <= M // 128]
        assert len(few) >= 6 and min(c.row_count for c in few) >= 64
        few = [c for pair in zip(few[::-1], few) for c in pair][:len(few)]
        rand = few + [c for c in rand if c.size > M // 128]
    elif order == "descending":
        rand = rand[::-1]
    table = type(classes)(*[L.gnnshap_class(size=c.size, full=c.full, row_count=c.row_count, weight=c.weight)
                            for c in full + rand])
    row = 0
    for c in table:
        c.row_begin = row
        row += c.row_count
    masks = torch.empty((plan.num_rows, plan.words_per_row), dtype=torch.int64, device=dev)
    weights = torch.empty(plan.num_rows, device=dev)
    ws = torch.empty(max(L.gnnshap_sample_workspace(plan), 256), dtype=torch.uint8, device=dev)
    L.gnnshap_sample_coalitions(plan, table, _vp(masks), _vp(weights), _vp(ws), ws.numel(),
                                torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    mb = sampler.unpack(masks_np(masks), M)
    sizes = np.concatenate([np.full(c.row_count, c.size) for c in table])
    np.testing.assert_array_equal(mb[:plan.num_rows // 2].sum(1), sizes)
    w = weights.cpu().numpy().astype(np.float64)
    v, f0, f1 = _game(M, mb, 3)
    yv = v(mb).astype(np.float32)
    fef = np.array([f0, f1], np.float32)
    phi, info = _solve(dev, plan, table, masks, torch.tensor(yv, device=dev), torch.tensor(fef, device=dev))
    assert info == 0
    _check_projected(phi, mb, w, yv, fef)


def _check_projected(phi, mb, w, yv, fef):
    """phi against the exact solution of the projected normal equations:
    |psi - psi*|_2 <= 1e-6 |b| / lambda_min, the iteration's tolerance, plus
    fp32 roundings."""
    M = mb.shape[1]
    delta = float(fef[1]) - float(fef[0])
    P = mb - mb.mean(1, keepdims=True)
    A = (P * w[:, None]).T @ P
    b = P.T @ (w * (yv.astype(np.float64) - float(fef[0]) - delta / M * mb.sum(1)))
    S = A + A.trace() / M * np.full((M, M), 1.0 / M)
    ref = delta / M + np.linalg.solve(S, b)
    bound = 1e-6 * np.linalg.norm(b) / np.linalg.eigvalsh(S)[0] + 1e-6 * np.linalg.norm(ref)
    assert np.linalg.norm(phi - ref) <= bound, (np.linalg.norm(phi - ref), bound)


@pytest.mark.parametrize("M", [700, 5003])
def test_a_solve_that_breaks_down_leaves_its_iterate(dev, M):
    """A negative weight of the random rows (no enumerated class) makes the
    operator negative definite: the first step has no positive curvature, in
    every workgroup.  info says so, and phi is the iterate as it was, Delta / M
    for every player, whichever workgroups run when the first one finds it."""
    plan, classes = L.gnnshap_plan_samples(M, 40000 if M > 5000 else 400, 3, 4)
    assert plan.random_begin == 0
    plan.iterative_threshold = 1
    masks = torch.empty((plan.num_rows, plan.words_per_row), dtype=torch.int64, device=dev)
    weights = torch.empty(plan.num_rows, device=dev)
    ws = torch.empty(max(L.gnnshap_sample_workspace(plan), 256), dtype=torch.uint8, device=dev)
    L.gnnshap_sample_coalitions(plan, classes, _vp(masks), _vp(weights), _vp(ws), ws.numel(),
                                torch.cuda.current_stream().cuda_stream)
    plan.random_weight = -1e-4
    for c in classes:
        c.weight = plan.random_weight
    g = torch.Generator(device=dev)
    g.manual_seed(1)
    y = torch.randn(plan.num_rows, generator=g, device=dev)
    fef = torch.tensor([0.25, 3.0], device=dev)
    want = np.float32((3.0 - 0.25) / M)
    for turn in range(20):
        print("breakdown", M, turn, flush=True)
        phi, info = _solve(dev, plan, classes, masks, y, fef)
        assert info == M + 1
        assert np.all(phi.astype(np.float32) == want)


@pytest.mark.parametrize("negative", ["random", "enumerated"])
def test_weights_of_either_sign(dev, negative):
    """A negative weight of the random or of the enumerated rows whose operator
    stays positive definite: phi against the exact solution of the projected
    normal equations."""
    M, p = 300, 12000
    print("weights", negative, flush=True)
    plan, classes, masks, _ = sample_on_gpu(M, p, 5, 6)
    plan.iterative_threshold = 1
    mb, _ = _oracle_rows(plan, masks, 5, 6)
    half = plan.num_rows // 2
    in_full = np.arange(half) < plan.random_begin
    in_full = np.concatenate([in_full, in_full])
    assert 0 < plan.random_begin < half
    P = mb - mb.mean(1, keepdims=True)
    full = np.linalg.eigvalsh(P[in_full].T @ P[in_full])
    rand = np.linalg.eigvalsh(P[~in_full].T @ P[~in_full])
    if negative == "random":       # half the enumerated part at its largest eigenvalue
        w_full, w_rand = 1.0, -0.5 * full[-1] / rand[-1]
    else:                          # (rand[0] = 0: the vector of ones, which P takes out)
        w_full, w_rand = -0.5 * rand[1] / full[-1], 1.0
    plan.random_weight = w_rand
    for c in classes:
        c.weight = w_full if c.full else w_rand
    v, f0, f1 = _game(M, mb, 11)
    yv = v(mb).astype(np.float32)
    fef = np.array([f0, f1], np.float32)
    phi, info = _solve(dev, plan, classes, masks, torch.tensor(yv, device=dev), torch.tensor(fef, device=dev))
    assert info == 0
    _check_projected(phi, mb, np.where(in_full, w_full, w_rand), yv, fef)
