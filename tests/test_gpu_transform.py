"""X W on split bf16 matrix products, against float64: tile edges in rows,
columns and K, rows whose start is not 16-byte aligned, the same bits for any
number of rows, a wide range of magnitudes, infinities, NaN and values that
round to infinity in bf16."""
import numpy as np
import pytest
import torch

from paper_2401_04829_amd import _lib as L
from paper_2401_04829_amd.explainer import _vp
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


def _transform(X, W):
    Z = torch.full((X.shape[0], W.shape[1]), -7.0, device=X.device)
    L.gnnshap_transform_features(_vp(X), X.shape[0], X.shape[1], _vp(W), W.shape[1], _vp(Z),
                                 torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return Z


@pytest.mark.parametrize("n,d,h", [(16384, 32, 64), (32700, 33, 40), (16385, 602, 128), (32641, 97, 65),
                                   (16384, 64, 129), (20001, 31, 64), (32895, 130, 127), (1000, 70, 48)])
def test_transform_against_float64(dev, n, d, h):
    print("transform", n, d, h, flush=True)
    g = torch.Generator(device=dev)
    g.manual_seed(n)
    X = torch.randn((n, d), generator=g, device=dev) * torch.exp(3 * torch.randn((n, 1), generator=g, device=dev))
    W = torch.randn((d, h), generator=g, device=dev) * torch.exp(3 * torch.randn((1, h), generator=g, device=dev))
    Z = _transform(X, W).double()
    exact = X.double() @ W.double()
    # fp32 products and sums: d roundings of at most 2^-24 of the sum of magnitudes
    bound = (d + 4) * 2.0 ** -24 * (X.double().abs() @ W.double().abs())
    assert bool(((Z - exact).abs() <= bound).all()), float(((Z - exact).abs() / bound).max())


# one row to the largest of each form: 16 x 64 outputs per workgroup (up to 159,
# 383 or 767 tiles of 128 x 64), 128 x 64 and 128 x 128; K of one step and a
# part, less than, exactly and more than the eight steps of one turn
@pytest.mark.parametrize("n,d,h", [(1, 128, 64), (15, 33, 48), (16, 257, 65), (17, 255, 112), (300, 602, 128),
                                   (301, 289, 250), (10112, 64, 128), (10113, 63, 128), (20353, 64, 64),
                                   (12160, 256, 200), (12289, 250, 256), (24449, 130, 128), (24577, 130, 128),
                                   (32769, 128, 66), (98177, 70, 48), (98176, 70, 48)])
def test_split_products_at_tile_edges(dev, n, d, h):
    print("split product", n, d, h, flush=True)
    g = torch.Generator(device=dev)
    g.manual_seed(n + d)
    X = torch.randn((n, d), generator=g, device=dev)
    W = torch.randn((d, h), generator=g, device=dev)
    Z = _transform(X, W).double()
    exact = X.double() @ W.double()
    bound = (d + 4) * 2.0 ** -24 * (X.double().abs() @ W.double().abs())
    worst = float(((Z - exact).abs() / bound).max())
    assert worst <= 1.0


@pytest.mark.parametrize("n,d,h", [(3000, 64, 64), (3000, 128, 128), (7000, 256, 256), (40000, 256, 128),
                                   (40000, 602, 128)])
def test_errors_of_split_products_have_no_direction(dev, n, d, h):
    """Results of either sign: the mean error over all of them, in their rms.
    The roundings (1e-7 each) leave 3e-10 over 192,000 and more; an odd number
    of steps of 32 leaves what one step drops, a quarter of 2^-24 of its own
    sum: 1.5e-8 / sqrt(19) at 602.  Steps that all drop the same way leave
    7.9e-9 (two steps) to 2.7e-8 (nineteen)."""
    print("mean error", n, d, h, flush=True)
    g = torch.Generator(device=dev)
    g.manual_seed(n + d)
    X = torch.randn((n, d), generator=g, device=dev)
    W = torch.randn((d, h), generator=g, device=dev)
    exact = X.double() @ W.double()
    err = (_transform(X, W).double() - exact) / exact.pow(2).mean().sqrt()
    assert float(err.pow(2).mean().sqrt()) <= 1.2e-7
    assert abs(float(err.mean())) <= 4e-9, float(err.mean())


@pytest.mark.parametrize("n,d,h", [(301, 1025, 128), (17, 1300, 66), (25000, 1030, 100), (33000, 1100, 128),
                                   (33025, 1027, 66), (98177, 300, 64), (301, 600, 64)])
def test_split_products_in_turns(dev, n, d, h):
    """Sums of several turns of eight steps, in every form: against float64, and
    rows alone against the same rows among all."""
    print("turns", n, d, h, flush=True)
    g = torch.Generator(device=dev)
    g.manual_seed(n + d)
    X = torch.randn((n, d), generator=g, device=dev)
    W = torch.randn((d, h), generator=g, device=dev)
    Z = _transform(X, W)
    exact = X.double() @ W.double()
    bound = (d + 4) * 2.0 ** -24 * (X.double().abs() @ W.double().abs())
    assert float(((Z.double() - exact).abs() / bound).max()) <= 1.0
    for i, k in ((0, 1), (n // 2, 17 if n > 40 else 3), (n - 16, 16)):
        assert torch.equal(_transform(X[i:i + k].contiguous(), W).view(torch.int32), Z[i:i + k].view(torch.int32))


@pytest.mark.parametrize("d,h,share,bound", [(1433, 128, 0.013, 7.2e-8), (1433, 128, 0.1, 1.0e-7),
                                             (1433, 64, 0.013, 7.2e-8), (500, 64, 0.1, 7.6e-8),
                                             (602, 128, 1.0, 1.0e-7)])
def test_rounding_of_sparse_rows(dev, d, h, share, bound):
    """Rows of which a share is not zero (ones, or log-normal values where there
    are more): rms error in rms of the results.  Bounds: halfway between the
    steps in turns (6.4e-8, 8.0e-8, 6.4e-8, 7.0e-8) and in one chain (7.9e-8,
    1.26e-7, 7.9e-8, 8.3e-8); dense rows, one chain: 9.2e-8."""
    print("sparse rows", d, h, share, flush=True)
    g = torch.Generator(device=dev)
    g.manual_seed(d + h)
    n = 2708
    X = torch.ones((n, d), device=dev) if share < 0.05 else torch.randn((n, d), generator=g, device=dev)
    if 0.05 < share < 1.0:
        X = torch.exp(X)
    X = X * (torch.rand((n, d), generator=g, device=dev) < share)
    W = (torch.rand((d, h), generator=g, device=dev) * 2 - 1) * (6 / (d + h)) ** 0.5
    exact = X.double() @ W.double()
    err = (_transform(X, W).double() - exact).pow(2).mean().sqrt() / exact.pow(2).mean().sqrt()
    assert float(err) <= bound, float(err)


@pytest.mark.parametrize("n,d,h", [(60000, 602, 128), (40000, 33, 48), (100000, 100, 64), (90000, 130, 100),
                                   (30000, 256, 256), (40000, 602, 41), (40000, 20, 64), (40000, 200, 32)])
def test_rows_do_not_depend_on_their_number(dev, n, d, h):
    """A row's bits are the same alone, among few and among all rows, and
    wherever it stands among them."""
    print("rows of", n, d, h, flush=True)
    g = torch.Generator(device=dev)
    g.manual_seed(n + h)
    X = torch.randn((n, d), generator=g, device=dev)
    W = torch.randn((d, h), generator=g, device=dev)
    Z = _transform(X, W)
    for a, b in ((7, 8), (0, 300), (n - 1001, n), (5, 13005), (100, 30000)):
        assert torch.equal(_transform(X[a:b], W), Z[a:b]), (a, b)


@pytest.mark.parametrize("ex,ew", [(0, 0), (-100, 20), (-115, 60), (-123, 99), (40, -123), (-60, -60), (60, -110),
                                   (110, -100), (-125, 116), (50, 50)])
def test_transform_at_the_ends_of_the_range(dev, ex, ew):
    """Operands of 2^ex and 2^ew times numbers of order one, rows and columns
    16 binades wide: down to the smallest normal fp32 numbers and below (the
    exact result is that of the fp32 values as they are), and sums of up to
    2^101, beyond those that the split product holds.  Bound: d roundings of
    at most 2^-24 of the sum of magnitudes, results below 2^-126 half an ulp
    of theirs besides."""
    n, d, h = 16500, 128, 128
    print("transform at", ex, ew, flush=True)
    g = torch.Generator(device=dev)
    g.manual_seed(ex * 300 + ew)
    pow2 = lambda shape: torch.randint(-8, 8, shape, generator=g, device=dev).double()
    X = (torch.randn((n, d), generator=g, device=dev).double() * 2.0 ** (ex + pow2((n, 1)))).float()
    W = (torch.randn((d, h), generator=g, device=dev).double() * 2.0 ** (ew + pow2((1, h)))).float()
    Z = _transform(X, W).double()
    exact = X.double() @ W.double()
    bound = (d + 4) * 2.0 ** -24 * (X.double().abs() @ W.double().abs()) + 2.0 ** -150
    worst = float(((Z - exact).abs() / bound).max())
    assert worst <= 1.0


def test_transform_special_values(dev):
    """Infinities, NaN and values above the largest bf16 number give what
    fp32 arithmetic gives; the other rows are untouched by them."""
    n, d, h = 16384, 64, 64
    X = torch.ones((n, d), device=dev)
    W = torch.full((d, h), 0.5, device=dev)
    W[3, 5] = 0.0
    X[10, 3] = float("inf")
    X[20, 4] = float("nan")
    X[30, 7] = 3.4e38
    X[40, 8], X[40, 9] = float("inf"), float("-inf")
    Z = _transform(X, W).cpu().numpy()
    want = np.full((n, h), 32.0, np.float32)
    want[:, 5] = 31.5
    want[10] = np.inf
    want[10, 5] = np.nan
    want[20] = np.nan
    want[30] = 1.7e38
    want[40] = np.nan
    np.testing.assert_allclose(Z, want, rtol=1e-6, equal_nan=True)
