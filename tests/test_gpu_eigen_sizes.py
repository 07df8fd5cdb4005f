"""gl_second_eigenpair at the edges of its row tiles (256 and 1024 rows; the
larger ones beyond 32 768 rows, where the tiles' sums are added by a launch of
their own beyond 131 072), and at Krylov sizes that fill and overfill a group
of 32 vectors, on rows of cliques."""

import math

import numpy as np
import pytest
import torch

import paper_2303_14495_amd as gl
from tests.gpu_helpers import DEV, say

pytestmark = pytest.mark.gpu


def _star_of_cliques(groups, size):
    """`groups` cliques of `size` nodes, consecutive cliques joined by one edge: CSR on the GPU."""
    n = groups * size
    i, j = torch.triu_indices(size, size, 1, device=DEV)
    base = torch.arange(groups, device=DEV)[:, None] * size
    a, b = (base + i).reshape(-1), (base + j).reshape(-1)
    a = torch.cat([a, torch.arange(groups - 1, device=DEV) * size])
    b = torch.cat([b, torch.arange(1, groups, device=DEV) * size])
    key, _ = torch.sort(torch.cat([a * n + b, b * n + a]))
    row = key // n
    rp = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rp[1:] = torch.cumsum(torch.bincount(row, minlength=n), 0)
    return rp, (key - row * n).to(torch.int32), torch.ones(key.numel(), dtype=torch.float64, device=DEV)


# two cliques joined by one edge: n and the Krylov size vary, one restart at most is needed
@pytest.mark.parametrize("n,krylov", [(4, 2), (254, 31), (256, 32), (258, 33), (1022, 34), (1026, 65)])
def test_two_cliques_against_dense(n, krylov):
    rp, col, w = _star_of_cliques(2, n // 2)
    op = gl.Operator(rp, col, w, store_w="f32")
    g = torch.Generator(device=DEV)
    g.manual_seed(n)
    lam, v, res, _ = op.second_eigenpair(torch.randn(n, generator=g, device=DEV), krylov=krylov, max_restarts=40, tol=1e-5)
    A = torch.zeros(n, n, dtype=torch.float64)
    row = torch.repeat_interleave(torch.arange(n), (rp[1:] - rp[:-1]).cpu())
    A[row, col.cpu().long()] = 1.0
    d = A.sum(1)
    ev, vec = torch.linalg.eigh(torch.eye(n, dtype=torch.float64) - A / (d.sqrt()[:, None] * d.sqrt()[None, :]))
    want = vec[:, 1].numpy()
    say(f"two cliques n={n} krylov={krylov}: lambda2 {lam:.8e} (want {float(ev[1]):.8e}) residual {res:.1e}")
    assert res <= 1e-5
    # |sin angle| <= residual / gap, eigenvalue error <= residual
    assert abs(lam - float(ev[1])) <= 1e-5
    assert 1 - abs(float(v.cpu().double().numpy() @ want)) <= max(1e-6, 2 * (1e-5 / float(ev[2] - ev[1])) ** 2)


@pytest.mark.parametrize("groups", [4096, 4097, 16384, 16400])
def test_row_tiles_residual(groups):
    """Many small cliques in a row (32 768, 32 776, 131 072 and 131 200 nodes): the
    returned vector is a unit vector, orthogonal to the null vector, and its
    Rayleigh quotient and residual in float64 are the reported ones."""
    rp, col, w = _star_of_cliques(groups, 8)
    n = groups * 8
    op = gl.Operator(rp, col, w, store_w="f32")
    g = torch.Generator(device=DEV)
    g.manual_seed(groups)
    lam, v, res, _ = op.second_eigenpair(torch.randn(n, generator=g, device=DEV), krylov=40, max_restarts=0, tol=1e-5)
    d = (rp[1:] - rp[:-1]).double()
    row = torch.repeat_interleave(torch.arange(n, device=DEV), rp[1:] - rp[:-1])
    x = v.double()
    y = x - torch.zeros_like(x).index_add_(0, row, x[col.long()] / (d[row] * d[col.long()]).sqrt())
    z = d.sqrt() / d.sqrt().norm()
    say(f"cliques n={n}: lambda {lam:.6e}, residual {res:.3e}")
    assert abs(float(x.norm()) - 1) <= 1e-6
    assert abs(float(x @ z)) <= 1e-5
    # f32 vectors and products: 2^-24 per entry of unit vectors, a few of them
    assert abs(float(x @ y) - lam) <= 2e-6
    assert abs(float((y - lam * x).norm()) - res) <= 2e-6
    assert float(v[v.abs().argmax()]) > 0
