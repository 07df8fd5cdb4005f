"""gl_power_max_eig from start vectors whose products stay far below the largest
eigenvalue, or only get there after some products: the iterates neither vanish
nor overflow between two normalisations."""

import numpy as np
import pytest
import torch

import paper_2303_14495_amd as gl
from tests.gpu_helpers import DEV, say

pytestmark = pytest.mark.gpu


def _path_and_star(joined, ratio, n=400, leaves=30):
    """A path of n nodes with weights 1 and a star with weights `ratio`, apart or joined at node `joined`."""
    A = np.zeros((n + leaves + 1, n + leaves + 1))
    i = np.arange(n - 1)
    A[i, i + 1] = 1.0
    A[n, n + 1:] = ratio
    if joined is not None:
        A[joined, n] = 1.0
    return A + A.T


def _operator(A, laplacian):
    i, j = np.nonzero(A)
    rp = np.zeros(A.shape[0] + 1, np.int64)
    rp[1:] = np.cumsum(np.bincount(i, minlength=A.shape[0]))
    return gl.Operator(*[torch.from_numpy(v).to(DEV) for v in (rp, j.astype(np.int32), A[i, j])], store_w="f32",
                       laplacian=laplacian)


# apart: the path's own largest eigenvalue; joined far away: the star is not reached; joined
# near: its eigenvalue, `ratio` times larger, takes over after 10 products
@pytest.mark.parametrize("joined", [None, 300, 10])
@pytest.mark.parametrize("ratio", [2.0**3, 2.0**12, 2.0**20, 2.0**40])
@pytest.mark.parametrize("iters", [1, 2, 17, 40, 150])
def test_start_away_from_the_largest(joined, ratio, iters):
    A = _path_and_star(joined, ratio)
    L = np.diag(A.sum(1)) - A
    x0 = np.zeros(A.shape[0], np.float32)
    x0[:5] = [1.0, -0.5, 0.25, -1.0, 0.5]
    x = x0.astype(np.float64)
    for _ in range(iters):
        x = L @ x
        x /= np.linalg.norm(x)
    want = x @ L @ x
    rq, _ = _operator(A, "unnormalized").power_max_eig(torch.from_numpy(x0).to(DEV), iters=iters)
    say(f"power joined={joined} ratio {ratio:g} after {iters}: {rq:.8e} (want {want:.8e})")
    # weights and vectors exact or rounded to 2^-24 per product of rows of at most 31 terms;
    # the star's share grows by a factor per product that is right to the same
    assert rq == pytest.approx(want, rel=2e-5)


@pytest.mark.parametrize("scale", [1.0, 2.0**40, 2.0**-20])
def test_smooth_start(scale):
    """A start vector near the null vector of a long path: the first products shrink it by 1e-4 and more."""
    A = _path_and_star(None, 1.0, n=2000, leaves=1) * scale
    L = np.diag(A.sum(1)) - A
    x0 = np.zeros(A.shape[0], np.float32)
    x0[:2000] = np.cos(np.pi * (np.arange(2000) + 0.5) / 2000)
    rq, lam = _operator(A, "unnormalized").power_max_eig(torch.from_numpy(x0).to(DEV), iters=60)
    say(f"smooth start x {scale:g}: {rq / scale:.4e}")
    # rounding of the products brings the upper spectrum in; what comes out is finite and within it
    assert 0.0 < rq <= 4.0 * scale * (1 + 1e-6) and lam <= 4.0 * scale * (1 + 1e-6)
