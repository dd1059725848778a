"""The wavefront sampler against the sequential algorithm, row by row.

It takes the steps of a random row 64 at a time and resolves by hand those
that meet: equal draws in a chunk, draws of another step's own player.  Just
above the one-lane-per-row limit (512 players) a chunk has several of either
kind; the players cover every position of a chunk's first player in its
32-bit word, and the last sizes the ends of the range.
"""
import numpy as np
import pytest

from oracle import sampler
from tests.gpu_util import masks_np, require_gpu, sample_on_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


@pytest.mark.parametrize("M,p", [(513, 3000), (514, 3000), (543, 2000), (544, 2000), (545, 2000), (575, 2000),
                                 (576, 2000), (577, 2000), (640, 2000), (767, 2000), (1025, 2000), (2047, 4000)])
def test_rows_equal_sequential_algorithm(dev, M, p):
    pl = sampler.plan(M, p)
    _, _, masks, weights = sample_on_gpu(M, p, 0xA5A5 + M, M)
    ref_m, ref_w = sampler.sample(pl, 0xA5A5 + M, M)
    np.testing.assert_array_equal(masks_np(masks), sampler.pack(ref_m))
    np.testing.assert_array_equal(weights.cpu().numpy(), ref_w.astype(np.float32))


@pytest.mark.parametrize("M", [65536, 131072])
def test_largest_player_sets(dev, M):
    p = 3 * M
    pl = sampler.plan(M, p)
    k = pl["k"]
    _, _, masks, _ = sample_on_gpu(M, p, 11, M)
    got = masks_np(masks)
    rows = np.unique(np.concatenate([np.random.default_rng(M).integers(0, k, 4), [k // 2 - 1, k - 1]]))
    ref_m, _ = sampler.sample_rows(pl, rows, 11, M)
    np.testing.assert_array_equal(got[rows], sampler.pack(ref_m))
