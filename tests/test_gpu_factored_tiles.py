"""The factored systems at the edges of their tiles: players around the 64-wide
count tiles, the 128-wide panels and the 256-row triangular segments; row words
around the 4 and 16 that one step and one stage of the counts take."""
import numpy as np
import pytest
import torch

from tests.gpu_util import require_gpu, sample_on_gpu
from tests.test_gpu_iterative import _game, _oracle_rows, _solve

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


@pytest.mark.parametrize("M,p", [(15, 510), (16, 128), (31, 640), (33, 2050), (63, 2048), (64, 2176), (65, 4096),
                                 (129, 3970), (193, 6000), (449, 2500), (511, 4100), (512, 5000), (513, 4098),
                                 (577, 6146), (705, 5000), (769, 8200), (1025, 9000)])
def test_factored_systems_at_tile_edges(dev, M, p):
    """phi against the projected normal equations on the oracle's rows: the
    exact solution, and the residual.  Bounds: a Cholesky solution in precision
    u has a backward error of at most about 3 M u (Higham, Accuracy and
    Stability of Numerical Algorithms, Thm 10.3), its effect on psi that times
    the condition number; and of a few sqrt(M) u as roundings fall (Higham and
    Mary, SIAM J. Sci. Comput. 41, 2019), four of which the residual is held
    to, relative to |S| |phi|.  The counts are whole numbers and add nothing: a
    single pair miscounted by one is 1 / (kr sqrt(M) / 4) of |S| |phi| and
    above that bound at every size here."""
    print("factored tiles", M, p, flush=True)
    plan, classes, masks, _ = sample_on_gpu(M, p, 5, 6)
    mb, w = _oracle_rows(plan, masks, 5, 6)
    v, f0, f1 = _game(M, mb, 3 * M)
    yv = v(mb).astype(np.float32)
    fef = np.array([f0, f1], np.float32)
    phi, info = _solve(dev, plan, classes, masks, torch.tensor(yv, device=dev), torch.tensor(fef, device=dev))
    delta = float(fef[1]) - float(fef[0])
    P = mb - mb.mean(1, keepdims=True)
    A = (P * w[:, None]).T @ P
    b = P.T @ (w * (yv.astype(np.float64) - float(fef[0]) - delta / M * mb.sum(1)))
    S = A + A.trace() / M * np.full((M, M), 1.0 / M)
    lam = np.linalg.eigvalsh(S)
    assert lam[0] > 1e-3 * lam[-1]   # the rows determine psi
    ref = delta / M + np.linalg.solve(S, b)
    assert info == 0
    bound = (3 * M * 2.0 ** -24 * lam[-1] / lam[0] + 1e-6) * np.linalg.norm(ref)
    assert np.linalg.norm(phi - ref) <= bound, (np.linalg.norm(phi - ref), bound)
    residual = np.linalg.norm(S @ (phi - phi.mean()) - b)
    assert residual <= 4 * M ** 0.5 * 2.0 ** -24 * lam[-1] * np.linalg.norm(phi)
