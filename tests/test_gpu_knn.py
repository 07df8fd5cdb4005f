"""GPU parity of gl_knn against the float64 brute-force oracle.

The kernel ranks by f32 distances, the oracle by f64, so near-ties may be
ordered differently: what is unique is compared exactly (index sets wherever
the k-th and (k+1)-th oracle distances are clearly apart, the distance lists
within f32 rounding), and everything else is checked for validity (distinct,
in range, not self, true distances equal to the oracle's k smallest).  On
integer lattices all distances are exact in f32 and the lists, ties included,
must match bitwise.
"""

import numpy as np
import pytest
import torch

import paper_2303_14495_amd as gl
from oracle import knn_oracle
from tests.gpu_helpers import DEV, say

pytestmark = pytest.mark.gpu


def mixture(n, d, seed):
    rng = np.random.default_rng(seed)
    means = 3.0 * rng.standard_normal((5, d))
    comp = rng.integers(0, 5, n)
    return (means[comp] + rng.standard_normal((n, d))).astype(np.float32)


def check(x, k, idx, d2, rows):
    """idx, d2: GPU results for the query rows `rows`."""
    n = x.shape[0]
    xd = x.astype(np.float64)
    oi, od = knn_oracle.knn(xd, k + 1, rows=rows)
    assert idx.shape == (len(rows), k)
    assert np.all((idx >= 0) & (idx < n))
    assert not np.any(idx == np.asarray(rows)[:, None])
    assert all(len(set(r)) == k for r in idx.tolist())
    # true distances of the chosen points
    true = ((xd[np.asarray(rows)][:, None, :] - xd[idx]) ** 2).sum(-1)
    scale = 1.0 + od[:, k - 1:k]
    tol = 4e-6 * scale * max(1, x.shape[1] // 8)
    assert np.all(np.diff(d2, axis=1) >= 0)
    assert np.all(np.abs(d2 - true) <= tol)
    assert np.all(np.abs(np.sort(true, axis=1) - od[:, :k]) <= tol)
    clear = (od[:, k] - od[:, k - 1]) > 2 * tol[:, 0]
    same = [set(a) == set(b) for a, b in zip(idx.tolist(), oi[:, :k].tolist())]
    assert all(s for s, c in zip(same, clear) if c)
    return float(np.mean(clear))


@pytest.mark.parametrize("d,k", [(1, 3), (3, 10), (10, 20), (16, 32), (27, 20), (40, 8), (64, 16)])
def test_knn_matches_oracle(d, k):
    n = 3000  # 11 full tiles of 256 plus a ragged tail
    x = mixture(n, d, seed=d * 100 + k)
    say(f"knn n={n} d={d} k={k}")
    idx, d2 = gl.knn(torch.from_numpy(x).to(DEV), k)
    torch.cuda.synchronize()
    frac = check(x, k, idx.cpu().numpy(), d2.cpu().numpy(), np.arange(n))
    assert frac > 0.25  # dense 1-D data has many near-ties; the rest must be clear


def test_knn_lattice_ties_exact():
    h, w = 40, 37
    yy, xx = np.mgrid[0:h, 0:w]
    pts = np.stack([yy.ravel(), xx.ravel()], 1).astype(np.float32)
    k = 12
    idx, d2 = gl.knn(torch.from_numpy(pts).to(DEV), k)
    oi, od = knn_oracle.knn(pts.astype(np.float64), k)
    assert np.array_equal(idx.cpu().numpy(), oi)
    assert np.array_equal(d2.cpu().numpy().astype(np.float64), od)


def test_knn_large_sampled():
    """Full served-size graph (n = 10^6, d = 10, k = 20): sampled rows
    against the oracle computed for those rows alone."""
    n, d, k = 1_000_000, 10, 20
    x = mixture(n, d, seed=11)
    say(f"knn n={n} d={d} k={k}")
    idx, d2 = gl.knn(torch.from_numpy(x).to(DEV), k)
    torch.cuda.synchronize()
    rows = np.random.default_rng(0).choice(n, 48, replace=False)
    rows = np.concatenate([rows, [0, n - 1]])
    check(x, k, idx.cpu().numpy()[rows], d2.cpu().numpy()[rows], rows)


def test_knn_minimum_and_nonfinite():
    x = np.array([[0.0], [1.0], [3.0], [np.nan], [7.0]], dtype=np.float32)
    idx, d2 = gl.knn(torch.from_numpy(x).to(DEV), 4)
    idx, d2 = idx.cpu().numpy(), d2.cpu().numpy()
    # finite points see the three other finite ones, then an unfilled slot
    assert list(idx[0]) == [1, 2, 4, -1] and np.isinf(d2[0, 3])
    assert list(idx[4]) == [2, 1, 0, -1]
    assert np.all(idx[3] == -1)
    # n = k + 1: every other point
    y = np.arange(6, dtype=np.float32)[:, None] * 2.0
    i2, _ = gl.knn(torch.from_numpy(y).to(DEV), 5)
    for r, row in enumerate(i2.cpu().numpy()):
        assert sorted(row) == [j for j in range(6) if j != r]


def test_knn_rejects_bad_sizes():
    x = torch.zeros((10, 3), device=DEV)
    for k in (0, 33, 10):
        with pytest.raises(gl.GLError):
            gl.knn(x, k)
    with pytest.raises(gl.GLError):
        gl.knn(torch.zeros((10, 4097), device=DEV), 3)


# The matrix-core path (d <= 64): edges of its dispatch.  Coordinates are small
# integers, so every distance is an exact f32 integer and the lists, ties to the
# lower index included, must equal the oracle's bit for bit.
#   d 4|5, 10|11, 15|16, 20|21, 31|32, 42|43: one k-step more;  k 4|5, 8|9, 12|13,
#   16|17, 20|21, 28|29: a longer list;  n: below, at and beyond a tile and a
#   workgroup of queries, one and several point segments.
@pytest.mark.parametrize("n,d,k,span", [
    (6000, 2, 4, 60), (6001, 4, 5, 12), (5856, 5, 8, 9), (5857, 10, 9, 6), (6015, 11, 12, 6), (6017, 15, 13, 6),
    (5000, 16, 16, 5), (4000, 20, 17, 5), (4001, 21, 20, 5), (3999, 31, 21, 4), (3000, 32, 28, 4), (3001, 42, 29, 4),
    (3002, 43, 32, 4), (2500, 64, 31, 4), (20000, 3, 10, 40), (65600, 3, 7, 200)])
def test_knn_matrix_path_exact(n, d, k, span):
    rng = np.random.default_rng(n + d)
    x = rng.integers(0, span, (n, d)).astype(np.float32)
    say(f"knn n={n} d={d} k={k} integers below {span}")
    idx, d2 = gl.knn(torch.from_numpy(x).to(DEV), k)
    rows = np.arange(n) if n <= 6100 else np.concatenate([np.arange(40), rng.choice(n, 400, replace=False), np.arange(n - 40, n)])
    oi, od = knn_oracle.knn(x.astype(np.float64), k, rows=rows)
    assert np.array_equal(idx.cpu().numpy()[rows], oi)
    assert np.array_equal(d2.cpu().numpy()[rows].astype(np.float64), od)


@pytest.mark.parametrize("n,shift,outlier", [(7000, 0.0, 0.0), (9000, 0.0, 0.0), (7000, 4096.0, 0.0), (7000, 0.0, 65536.0)])
def test_knn_every_query_rescanned(n, shift, outlier):
    """27 distinct places: every list is full of ties, so no query has a proof
    and all are scanned (one, and four, queries per wavefront); far from the
    origin, and with a point that sets the scale alone."""
    rng = np.random.default_rng(n)
    x = (rng.integers(0, 3, (n, 3)) + shift).astype(np.float32)
    x[5] += outlier
    k = 20
    idx, d2 = gl.knn(torch.from_numpy(x).to(DEV), k)
    rows = np.delete(np.arange(n), 5)  # the outlier's own distances exceed f32's integers
    oi, od = knn_oracle.knn(x.astype(np.float64), k, rows=rows)
    assert np.array_equal(idx.cpu().numpy()[rows], oi)
    assert np.array_equal(d2.cpu().numpy()[rows].astype(np.float64), od)


def test_knn_matrix_path_nonfinite_and_constant():
    n, k = 6000, 6
    x = np.random.default_rng(3).integers(0, 40, (n, 3)).astype(np.float32)
    x[17, 1], x[99, 0], x[1234, 2] = np.nan, np.inf, -np.inf
    ok = np.isfinite(x).all(1)
    idx, d2 = (t.cpu().numpy() for t in gl.knn(torch.from_numpy(x).to(DEV), k))
    back = np.flatnonzero(ok)
    oi, od = knn_oracle.knn(x[ok].astype(np.float64), k)
    assert np.array_equal(idx[ok], back[oi]) and np.array_equal(d2[ok].astype(np.float64), od)
    assert np.all(idx[~ok] == -1) and np.all(np.isinf(d2[~ok]))
    # all points alike: the lowest other indices, at distance 0
    idx, d2 = (t.cpu().numpy() for t in gl.knn(torch.full((n, 3), 2.5, device=DEV), k))
    assert np.all(d2 == 0.0)
    assert np.array_equal(idx[100], np.arange(k)) and np.array_equal(idx[2], [0, 1, 3, 4, 5, 6])


def test_knn_under_capture():
    """A captured call (scanned: it allocates nothing) on new contents at every replay."""
    n, d, k = 6500, 4, 8
    rng = np.random.default_rng(7)
    x = torch.zeros((n, d), device=DEV)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        idx, d2 = gl.knn(x, k)
    for _ in range(3):
        xi = rng.integers(0, 12, (n, d)).astype(np.float32)
        x.copy_(torch.from_numpy(xi))
        g.replay()
        torch.cuda.synchronize()
        ei, ed = gl.knn(x, k)
        assert torch.equal(idx, ei) and torch.equal(d2, ed)


# ---------------------------------------------------------------------------
# gl_knn_graph: union-symmetric graph with local-scaling weights
# ---------------------------------------------------------------------------

def _graph_gpu(idx, d2, scale_rank):
    rp, col, w = gl.knn_graph(torch.from_numpy(np.ascontiguousarray(idx)).to(DEV),
                              torch.from_numpy(np.ascontiguousarray(d2)).to(DEV), scale_rank)
    return rp.cpu().numpy(), col.cpu().numpy(), w.cpu().numpy()


@pytest.mark.parametrize("n,d,k,rank", [(1500, 6, 10, 7), (3000, 10, 20, 7), (257, 3, 1, 1)])
def test_knn_graph_assembly_matches_oracle(n, d, k, rank):
    """Same kNN lists on both sides (the oracle's, distances rounded to float32):
    the edge sets must be identical and the weights agree to rounding."""
    x = mixture(n, d, n + k).astype(np.float64)
    idx, d2 = knn_oracle.knn(x, k)
    d2f = d2.astype(np.float32)
    say(f"knn graph assembly n={n} k={k} rank={rank}")
    rp, col, w = _graph_gpu(idx.astype(np.int32), d2f, rank)
    orp, ocol, ow = knn_oracle.graph_from_knn(n, idx, d2f.astype(np.float64), rank)
    assert rp.tolist() == orp.tolist()
    assert col.tolist() == ocol.tolist()
    assert np.abs(w - ow).max() <= 1e-14 * max(1.0, ow.max())


def test_knn_graph_end_to_end_vs_oracle():
    """gl_knn (float32) then gl_knn_graph against the oracle's recipe in
    float64.  Rows whose k-th and (k+1)-th oracle neighbours are clearly apart
    must pick the oracle's list; near-tie rows may pick either point, so the
    oracle graph is built from the GPU's lists with float64 distances: the edge
    sets must then be identical and the weights agree to float32 rounding."""
    n, d, k, rank = 2000, 8, 12, 7
    x = mixture(n, d, 99)
    xd = x.astype(np.float64)
    oi, od = knn_oracle.knn(xd, k + 1)
    idx, d2 = gl.knn(torch.from_numpy(x).to(DEV), k)
    gi = idx.cpu().numpy()
    clear = (od[:, k] - od[:, k - 1]) / od[:, k] > 1e-5
    assert np.array_equal(gi[clear], oi[clear, :k])
    rp, col, w = gl.knn_graph(idx, d2, rank)
    rp, col, w = rp.cpu().numpy(), col.cpu().numpy(), w.cpu().numpy()
    true_d2 = ((xd[:, None, :] - xd[gi]) ** 2).sum(-1)
    orp, ocol, ow = knn_oracle.graph_from_knn(n, gi, true_d2, rank)
    assert rp.tolist() == orp.tolist() and col.tolist() == ocol.tolist()
    rel = np.abs(w - ow) / ow
    say(f"knn graph end to end: nnz {len(col)}, {int((~clear).sum())} near-tie rows, "
        f"max weight rel err {rel.max():.2e}")
    assert rel.max() <= 2e-4
    # the graph is a valid operator input, and the operator accepts it
    op = gl.Operator(torch.from_numpy(rp).to(DEV), torch.from_numpy(col).to(DEV),
                     torch.from_numpy(w).to(DEV), store_w="f32")
    assert op.info()["nnz"] == len(col)


def test_knn_graph_duplicates_and_errors():
    # four coincident points and one far away: zero scales take the floor,
    # coincident pairs get weight 1, the far point is isolated -> rejected
    x = np.array([[0.0], [0.0], [0.0], [0.0], [1e3]], dtype=np.float64)
    idx, d2 = knn_oracle.knn(x, 2)
    with pytest.raises(gl.GLError):
        _graph_gpu(idx.astype(np.int32), d2.astype(np.float32), 1)
    x = np.array([[0.0], [0.0], [0.0], [0.0], [1.0], [1.0], [1.0]], dtype=np.float64)
    idx, d2 = knn_oracle.knn(x, 3)
    rp, col, w = _graph_gpu(idx.astype(np.int32), d2.astype(np.float32), 1)
    orp, ocol, ow = knn_oracle.graph_from_knn(7, idx, d2, 1)
    assert rp.tolist() == orp.tolist() and col.tolist() == ocol.tolist()
    assert np.array_equal(w, ow)
    good_i = np.array([[1], [0], [1]], dtype=np.int32)
    good_d = np.ones((3, 1), dtype=np.float32)
    for bad_i, bad_d in [(np.array([[0], [0], [1]], np.int32), good_d),     # self
                         (np.array([[1], [3], [1]], np.int32), good_d),     # out of range
                         (good_i, np.array([[1], [-1], [1]], np.float32)),  # negative
                         (good_i, np.array([[1], [np.nan], [1]], np.float32))]:
        with pytest.raises(gl.GLError):
            _graph_gpu(bad_i, bad_d, 1)


def _lists_with_row(n, length):
    """Lists of 2 whose union gives point 5 a row of `length` entries before
    duplicates go: its own two and those of length - 2 points."""
    idx = np.empty((n, 2), np.int32)
    for i in range(n):
        ring = [j for j in ((i + s) % n for s in range(1, 5)) if j != 5]
        idx[i] = (5, ring[0]) if i != 5 and (i < length - 1) else (ring[0], ring[1])
    assert int((idx == 5).sum()) == length - 2
    return idx


@pytest.mark.parametrize("case", [63, 64, 65, 4096, 4097, 12290, "dense", "repeated"])
def test_knn_graph_row_lengths(case):
    """Rows at the edges of a wavefront (64 entries), of one sorted run (4096) and
    of several; lists of 70 (every row long); a point repeated within a list.
    Distances are a symmetric function of the pair and some weights vanish.
    The weight is one float64 division and exponential on both sides: 4 ulp."""
    rng = np.random.default_rng(7)
    if case == "dense":
        n = 300
        idx = np.stack([rng.permutation(np.delete(np.arange(n), i))[:70] for i in range(n)]).astype(np.int32)
    elif case == "repeated":
        n = 40
        idx = ((np.arange(n)[:, None] + rng.integers(1, 4, (n, 9))) % n).astype(np.int32)
    else:
        n = case + 30
        idx = _lists_with_row(n, case)
    i = np.arange(n)[:, None]
    lo, hi = np.minimum(i, idx).astype(np.int64), np.maximum(i, idx).astype(np.int64)
    d2 = (0.5 + (lo * 31 + hi * 17) % 97 / 64.0).astype(np.float32)
    d2[((lo + hi) % 13 == 0) & (hi - lo > 4)] = 1e5
    rank = idx.shape[1]
    say(f"knn graph rows {case}")
    rp, col, w = _graph_gpu(idx, d2, rank)
    orp, ocol, ow = knn_oracle.graph_from_knn(n, idx, d2.astype(np.float64), rank)
    assert rp.tolist() == orp.tolist()
    assert col.tolist() == ocol.tolist()
    assert np.all(np.abs(w - ow) <= 4 * np.spacing(ow))


# ---------------------------------------------------------------------------
# wide features (d > 64): f16 Gram matrix on the matrix cores, exact refine,
# certificate, exact rescan of uncertified rows
# ---------------------------------------------------------------------------

def _exact_f32(x, rows, idx):
    """Distances as the kernels form them: f32 fused multiply-adds in
    coordinate order (t^2 is exact in float64, one rounding per step)."""
    acc = np.zeros(idx.shape, dtype=np.float32)
    q = x[np.asarray(rows)][:, None, :]
    p = x[idx]
    for c in range(x.shape[1]):
        t = (q[..., c] - p[..., c]).astype(np.float32)
        acc = (acc.astype(np.float64) + t.astype(np.float64) ** 2).astype(np.float32)
    return acc


@pytest.mark.parametrize("n,d,k", [(3000, 65, 10), (3000, 100, 1), (2500, 784, 10), (2100, 300, 32)])
def test_knn_wide_matches_oracle(n, d, k):
    x = mixture(n, d, seed=d + k)
    say(f"wide knn n={n} d={d} k={k}")
    idx, d2 = gl.knn(torch.from_numpy(x).to(DEV), k)
    fb = gl.knn_fallback_rows()
    idx, d2 = idx.cpu().numpy(), d2.cpu().numpy()
    frac = check(x, k, idx, d2, np.arange(n))
    say(f"  clear rows {frac:.4f}, exact rescans {fb}")
    assert frac > 0.5  # concentrated distances in high dimension: many near-ties
    assert fb <= n // 20
    # the distances are the kernels' own f32 sums (up to the emulation's double rounding)
    ref = _exact_f32(x, np.arange(n), idx)
    assert np.abs(d2 - ref).max() <= 1e-6 * max(1.0, float(ref.max()))


@pytest.mark.parametrize("n,d,k", [(40, 70, 5), (129, 65, 12), (300, 128, 13), (1100, 192, 8)])
def test_knn_wide_block_edges(n, d, k):
    """Shapes at the edges of the fused kernel's blocking: fewer points than
    one 128-point block (one query block, a partial point block), one point
    past a block, d a multiple of the 64-coordinate staging step (no padding),
    and k on both sides of the switch between eight lists of 8 (k <= 12) and
    two lists of 32 candidates per query."""
    x = mixture(n, d, seed=n + d + k)
    say(f"wide knn edges n={n} d={d} k={k}")
    idx, d2 = gl.knn(torch.from_numpy(x).to(DEV), k)
    fb = gl.knn_fallback_rows()
    idx, d2 = idx.cpu().numpy(), d2.cpu().numpy()
    check(x, k, idx, d2, np.arange(n))
    say(f"  exact rescans {fb}")
    ref = _exact_f32(x, np.arange(n), idx)
    assert np.abs(d2 - ref).max() <= 1e-6 * max(1.0, float(ref.max()))


@pytest.mark.parametrize("n,d,k", [(255, 96, 10), (257, 97, 32), (768, 65, 12), (769, 127, 13), (1025, 160, 32),
                                   (16384, 65, 10), (16385, 96, 12), (17000, 70, 32)])
def test_knn_wide_plan_edges(n, d, k):
    """Points around the 256-point blocks and the 4 segments of a query block (every
    fourth point each below 769), lists of 8 for k <= 12 and of 12 above, coordinates around
    the 32 of a staging step, and query blocks around one full round of 64 (16384
    points: none left over, then one and three cut into 16 segments)."""
    x = mixture(n, d, seed=n + d + k)
    say(f"wide knn plan n={n} d={d} k={k}")
    idx, d2 = gl.knn(torch.from_numpy(x).to(DEV), k)
    fb = gl.knn_fallback_rows()
    idx, d2 = idx.cpu().numpy(), d2.cpu().numpy()
    rows = np.unique(np.concatenate([np.arange(0, n, max(1, n // 400)), np.arange(max(0, n - 40), n)]))
    check(x, k, idx[rows], d2[rows], rows)
    say(f"  exact rescans {fb}")
    assert fb <= n // 20
    ref = _exact_f32(x, rows, idx[rows])
    assert np.abs(d2[rows] - ref).max() <= 1e-6 * max(1.0, float(ref.max()))


def test_knn_wide_many_copies():
    """20 integer points, 100 copies of each: more points within the error bound of
    the k-th distance than a wavefront refines, so the rescan decides the ties."""
    rng = np.random.default_rng(3)
    x = np.repeat(rng.integers(0, 9, (20, 80)), 100, axis=0).astype(np.float32)
    x = x[rng.permutation(len(x))]
    idx, d2 = gl.knn(torch.from_numpy(x).to(DEV), 12)
    oi, od = knn_oracle.knn(x.astype(np.float64), 12)
    assert np.array_equal(idx.cpu().numpy(), oi)
    assert np.array_equal(d2.cpu().numpy(), od.astype(np.float32))


def test_knn_wide_ties_use_the_exact_rescan():
    """The 96 unit vectors of R^96 are all at squared distance 2 from each
    other: every candidate ties with points outside the 64 candidates, so
    those rows lose the certificate and are rescanned exactly; with other
    integer points (and duplicates) around, the result must equal the float64
    oracle exactly, ties to the lower index."""
    rng = np.random.default_rng(12)
    n, d, k = 1200, 96, 12
    x = rng.integers(0, 3, (n, d)).astype(np.float32) + 4.0
    x[:d] = np.eye(d, dtype=np.float32)
    x[300:360] = x[200:260]  # exact duplicates: distance-0 ties
    idx, d2 = gl.knn(torch.from_numpy(x).to(DEV), k)
    fb = gl.knn_fallback_rows()
    oi, od = knn_oracle.knn(x.astype(np.float64), k)
    say(f"wide knn ties: exact rescans {fb} of {n}")
    assert fb >= d
    assert np.array_equal(idx.cpu().numpy(), oi)
    assert np.array_equal(d2.cpu().numpy(), od.astype(np.float32))


def test_knn_wide_rejects_nonfinite():
    x = mixture(500, 80, seed=1)
    x[7, 3] = np.nan
    with pytest.raises(gl.GLError):
        gl.knn(torch.from_numpy(x).to(DEV), 5)
