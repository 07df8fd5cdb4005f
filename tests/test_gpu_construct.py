"""Graph checks and degrees by 16 lanes per row, and the power method's iterates
between two normalisations: the places where a group, a row or a run of products
ends."""

import numpy as np
import pytest
import torch

import paper_2303_14495_amd as gl
from tests.gpu_helpers import DEV, say

pytestmark = pytest.mark.gpu


def _band(n, half):
    """Every node joined to the `half` nodes on each side: CSR arrays with float64 weights."""
    rows = [[j for j in range(max(0, i - half), min(n, i + half + 1)) if j != i] for i in range(n)]
    rp = np.zeros(n + 1, np.int64)
    rp[1:] = np.cumsum([len(r) for r in rows])
    col = np.concatenate(rows).astype(np.int32)
    row = np.repeat(np.arange(n), np.diff(rp))
    w = 1.0 + 0.25 * ((row * 7 + col * 7) % 5)
    return rp, col, w


def _operator(rp, col, w, **kw):
    return gl.Operator(torch.from_numpy(rp).to(DEV), torch.from_numpy(col).to(DEV), torch.from_numpy(w).to(DEV), **kw)


# rows of 2 * half entries inside the band: a partial group, one, one and one entry, two, two and one entry
@pytest.mark.parametrize("n,half", [(40, 3), (53, 8), (200, 17), (130, 16), (257, 33)])
def test_one_defect_is_named(n, half):
    rp, col, w = _band(n, half)
    _operator(rp, col, w).close()
    i = n // 2
    length = int(rp[i + 1] - rp[i])
    for at in sorted({0, length // 2, min(15, length - 1), min(16, length - 1), length - 1}):
        p = int(rp[i]) + at
        for what, match in (("asymmetric", "symmetric"), ("weight", "weight"), ("range", "out of"), ("self", "self-loop"),
                            ("order", "increasing")):
            c2, w2 = col.copy(), w.copy()
            if what == "asymmetric":
                w2[p] = np.nextafter(w2[p], 9.0)
            elif what == "weight":
                w2[p] = 0.0
            elif what == "range":
                c2[p] = n
            elif what == "self":
                c2[p] = i
            else:
                if at == 0:
                    continue
                c2[p] = c2[p - 1]
            with pytest.raises(gl.GLError, match=match) as e:
                _operator(rp, c2, w2)
            # the first offending row is this one, or one of its neighbours where they miss their partner
            first = int(str(e.value).split("row ")[1].split(")")[0])
            assert abs(first - i) <= half, (what, at, first)
    r2 = rp.copy()
    r2[i] = r2[i + 1] + 1
    with pytest.raises(gl.GLError, match="row_ptr"):
        _operator(r2, col, w)
    with pytest.raises(gl.GLError, match="degree"):  # a row without entries
        _operator(np.concatenate([rp, rp[-1:]]), col, w)


@pytest.mark.parametrize("n,half", [(40, 3), (53, 8), (200, 17), (257, 33)])
@pytest.mark.parametrize("weight", [np.float64, np.float32])
def test_degrees_and_weights(n, half, weight):
    rp, col, w = _band(n, half)
    w = w.astype(weight)
    row = np.repeat(np.arange(n), np.diff(rp))
    deg = np.bincount(row, w.astype(np.float64), n)
    x = np.random.default_rng(n).uniform(-1, 1, (n, 2))
    ref = x.copy()
    np.subtract.at(ref, row, (w / (np.sqrt(deg[row]) * np.sqrt(deg[col])))[:, None] * x[col])
    y = _operator(rp, col, w, store_w="f64").laplacian_apply(torch.from_numpy(x).to(DEV)).cpu().numpy()
    assert np.abs(y - ref).max() <= 1e-14  # rows of up to 66 terms of at most 1


@pytest.mark.parametrize("iters", [0, 1, 15, 16, 17, 33])
@pytest.mark.parametrize("laplacian,factor", [("normalized", 1.0), ("unnormalized", 1.0), ("unnormalized", 2.0**60),
                                              ("unnormalized", 2.0**-60)])
def test_power_iterates(iters, laplacian, factor):
    """Rayleigh quotient after `iters` products, for weights of the size of 1, 2^60 and 2^-60."""
    n = 300
    rp, col, w = _band(n, 5)
    row = np.repeat(np.arange(n), np.diff(rp))
    deg = np.bincount(row, w, n)
    A = np.zeros((n, n))
    A[row, col] = w
    L = np.diag(deg) - A if laplacian == "unnormalized" else np.eye(n) - A / np.sqrt(deg[:, None] * deg[None, :])
    x0 = np.random.default_rng(1).uniform(-1, 1, n).astype(np.float32)
    x = x0.astype(np.float64)
    for _ in range(iters):
        x = L @ x
        x /= np.linalg.norm(x)
    want = x @ L @ x / (x @ x) * factor
    op = _operator(rp, col, w * factor, store_w="f32", laplacian=laplacian)
    rq, lam = op.power_max_eig(torch.from_numpy(x0).to(DEV), iters=iters)
    say(f"power {laplacian} x {factor:.0e} after {iters}: {rq:.8e} (want {want:.8e})")
    # f32 weights and vectors: 2^-24 per product and row of 10 terms, quadratic in the quotient but for the last product
    assert rq == pytest.approx(want, rel=2e-5)
    if laplacian == "normalized":
        assert lam == pytest.approx(min(2.0, 1.01 * rq))
