"""gl_second_eigenpair restarted until its tolerance: graphs whose largest degree
is far above the residual that is asked for, with both Laplacians, and graphs
with few distinct eigenvalues, whose Krylov space ends at once."""

import numpy as np
import pytest
import torch

import paper_2303_14495_amd as gl
from tests.gpu_helpers import DEV, say
from tests.test_gpu_eigen_sizes import _star_of_cliques

pytestmark = pytest.mark.gpu


def _csr(A):
    i, j = np.nonzero(A)
    rp = np.zeros(A.shape[0] + 1, np.int64)
    rp[1:] = np.cumsum(np.bincount(i, minlength=A.shape[0]))
    return [torch.from_numpy(v).to(DEV) for v in (rp, j.astype(np.int32), A[i, j])]


def _hub_and_band(n, hub):
    """Node 0 joined to the `hub` nodes behind it; the others joined to the three on each side."""
    A = np.zeros((n, n))
    A[0, 1:hub + 1] = 1.0
    for t in (1, 2, 3):
        i = np.arange(1, n - t)
        A[i, i + t] = 0.5
    return A + A.T


def _laplacian(A, laplacian):
    d = A.sum(1)
    return np.diag(d) - A if laplacian == "unnormalized" else np.eye(len(d)) - A / np.sqrt(np.outer(d, d))


def _solve(A, laplacian, seed, **kw):
    op = gl.Operator(*_csr(A), store_w="f32", laplacian=laplacian)
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return op.second_eigenpair(torch.randn(A.shape[0], generator=g, device=DEV), **kw)


# Residuals asked for are at least 5 times the float rounding of L v: 2^-24 d_i |v_i|
# over the rows, |v_hub| about n^-1/2 (1.9e-6 for the largest degree of 1199 times 1).
@pytest.mark.parametrize("laplacian,scale", [("unnormalized", 1.0), ("unnormalized", 2.0**10), ("unnormalized", 2.0**-10),
                                             ("normalized", 1.0)])
def test_restarts_reach_tolerance(laplacian, scale):
    A = _hub_and_band(1500, 1199)
    tol = 1e-5 * (scale if laplacian == "unnormalized" else 1.0)
    lam, v, res, rs = _solve(A * scale, laplacian, 1, krylov=24, max_restarts=60, tol=tol)
    L = _laplacian(A * scale, laplacian)
    want = np.linalg.eigvalsh(L)[1]
    x = v.cpu().double().numpy()
    real = float(np.linalg.norm(L @ x - lam * x))
    say(f"hub {laplacian} x {scale:g}: lambda {lam:.6e} (want {want:.6e}), residual {res:.2e} (f64 {real:.2e}), {rs} restarts")
    assert res <= tol
    assert abs(lam - want) <= tol  # an eigenvalue lies within the residual, and the second is the nearest
    assert real <= 2 * tol


def test_points_reach_tolerance():
    """kNN graph of two clouds, L = D - W, 16 Krylov vectors: 2e-6 times the largest degree is above the tolerance."""
    g = torch.Generator(device=DEV)
    g.manual_seed(4)
    x = torch.randn(4096, 2, generator=g, device=DEV)
    x[2048:] += 4
    rp, col, w = gl.knn_graph(*gl.knn(x, 15))
    op = gl.Operator(rp, col, w, store_w="f32", laplacian="unnormalized")
    lam, v, res, rs = op.second_eigenpair(torch.randn(4096, generator=g, device=DEV), krylov=16, max_restarts=60, tol=1e-5)
    say(f"points: lambda {lam:.6e}, residual {res:.2e}, {rs} restarts")
    assert res <= 1e-5


@pytest.mark.parametrize("laplacian", ["normalized", "unnormalized"])
@pytest.mark.parametrize("n,krylov", [(50, 49), (300, 40)])
def test_complete_graph_ends_at_once(laplacian, n, krylov):
    """One eigenvalue beside 0: the Krylov space is one vector, and restarts that change nothing end the loop."""
    lam, _, res, rs = _solve(np.ones((n, n)) - np.eye(n), laplacian, n, krylov=krylov, max_restarts=50, tol=1e-30)
    want = n if laplacian == "unnormalized" else n / (n - 1)
    say(f"K_{n} {laplacian}: lambda {lam:.8e}, residual {res:.1e}, {rs} restarts")
    # residual: rounding of L v, some 2^-24 of its unit rows of n terms of at most 1 (largest magnitudes first)
    assert abs(lam - want) <= 1e-5 * want and res <= 1e-5 * want


# 8192 row tiles of 1024 rows and one more: the tiles' norms are added up by every
# workgroup, or by a launch of their own
@pytest.mark.parametrize("groups", [1048576, 1048580])
def test_many_row_tiles(groups):
    rp, col, w = _star_of_cliques(groups, 8)
    n = groups * 8
    op = gl.Operator(rp, col, w, store_w="f32")
    g = torch.Generator(device=DEV)
    g.manual_seed(groups)
    lam, v, res, _ = op.second_eigenpair(torch.randn(n, generator=g, device=DEV), krylov=6, max_restarts=1, tol=1e-9)
    d = (rp[1:] - rp[:-1]).double()
    row = torch.repeat_interleave(torch.arange(n, device=DEV), rp[1:] - rp[:-1])
    x = v.double()
    y = x - torch.zeros_like(x).index_add_(0, row, x[col.long()] / (d[row] * d[col.long()]).sqrt())
    say(f"cliques n={n}: lambda {lam:.6e}, residual {res:.3e}")
    # f32 vectors and products: 2^-24 per entry of unit vectors, a few of them
    assert abs(float(x.norm()) - 1) <= 1e-6
    assert abs(float(x @ y) - lam) <= 2e-6
    assert abs(float((y - lam * x).norm()) - res) <= 2e-6
