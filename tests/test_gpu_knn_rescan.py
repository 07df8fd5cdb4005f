"""gl_knn for d <= 64 where queries have no proof, or the matrix cores are not used:
the scans of many queries, on both sides of the counts where a thread per query
takes over from a wavefront per query.  Coordinates are small whole numbers, so
every distance is an exact float32 integer and the lists, ties to the lower
index included, must equal the reference's."""

import numpy as np
import pytest
import torch

import paper_2303_14495_amd as gl
from tests.gpu_helpers import DEV, say

pytestmark = pytest.mark.gpu


def _points(n, d, tied, seed):
    """`tied` points in groups of 60 copies, the others with coordinates below 200."""
    rng = np.random.default_rng(seed)
    x = rng.integers(0, 200, (n, d)).astype(np.float32)
    x[:tied] = x[np.arange(tied) // 60]
    return torch.from_numpy(x[rng.permutation(n)]).to(DEV)


def _reference(x, k, rows):
    """Exact lists of the query rows: (distance, index) sorted as whole numbers, on the GPU in float64."""
    n = x.shape[0]
    xd = x.double()
    out_i, out_d = [], []
    for q in rows:
        dist = ((xd - xd[q]) ** 2).sum(1)
        key = torch.where(torch.isfinite(dist), dist, torch.full_like(dist, 2.0**40)).to(torch.int64) * n + torch.arange(n, device=DEV)
        key[q] = 2**62
        best = torch.sort(torch.topk(key, k, largest=False).values).values
        out_i.append(best % n)
        out_d.append(best // n)
    return torch.stack(out_i), torch.stack(out_d)


def _check(x, k, idx, d2, seed):
    n = x.shape[0]
    rows = sorted(set(np.random.default_rng(seed).choice(n, 60, replace=False).tolist() + [0, 63, 64, 255, 256, n - 2, n - 1]))
    rows = [q for q in rows if bool(torch.isfinite(x[q]).all())]
    want_i, want_d = _reference(x, k, rows)
    assert torch.equal(idx[rows].to(torch.int64), want_i)
    assert torch.equal(d2[rows].to(torch.int64), want_d)


# listed queries: the limits are 36 000 (d <= 16) and 28 000; k at the
# edges of the register lists (8, 16, 24, 32); d below, at and between the widths
@pytest.mark.parametrize("n,d,k,tied", [
    (37000, 2, 8, 35940), (37000, 3, 9, 36060), (36500, 4, 16, 35940), (36501, 7, 17, 36060), (36100, 16, 32, 36060),
    (49000, 2, 24, 48000),
    (28100, 17, 24, 28020), (28200, 20, 25, 28020), (28300, 21, 15, 27960), (29000, 27, 10, 28980), (28500, 33, 5, 28500),
    (28500, 41, 20, 28500), (28500, 49, 30, 28500), (28500, 57, 16, 28500), (28500, 64, 32, 28440), (30000, 64, 8, 600)])
def test_listed_queries(n, d, k, tied):
    say(f"knn n={n} d={d} k={k}, {tied} points in copies")
    x = _points(n, d, tied, n + d)
    idx, d2 = gl.knn(x, k)
    _check(x, k, idx, d2, d)


# every point: the limits are 110 000 (d <= 3 and k > 16), 50 000 (d <= 16) and 36 000; under
# capture, where nothing may be allocated, and with a coordinate that is no number
@pytest.mark.parametrize("n,d,k", [(110001, 1, 17), (109999, 3, 20), (50001, 3, 16), (49999, 10, 4), (50300, 15, 25),
                                   (36001, 17, 8), (35999, 27, 32), (36500, 40, 12), (36001, 64, 32)])
@pytest.mark.parametrize("capture", [False, True])
def test_every_point(n, d, k, capture):
    say(f"knn n={n} d={d} k={k} capture={capture}")
    x = _points(n, d, 6000, n + k)
    if capture:
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            idx, d2 = gl.knn(x, k)
        graph.replay()
        torch.cuda.synchronize()
    else:
        x[77, d - 1] = float("nan")
        idx, d2 = gl.knn(x, k)
        assert bool((idx[77] == -1).all()) and bool(torch.isinf(d2[77]).all())
        assert not bool((idx == 77).any())
    _check(x, k, idx, d2, k)


def _mixture(n, d, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    means = 3.0 * torch.randn(5, d, generator=g, device=DEV)
    return means[torch.randint(0, 5, (n,), generator=g, device=DEV)] + torch.randn(n, d, generator=g, device=DEV)


# one case per k-step count and list length of the matrix path, and several segments.
# The error bound is about 4e-5 |q|^2 at d = 64 and 3e-6 |q|^2 at d = 2; the T-th of a
# query's approximate distances lies at least 4 places behind the k-th, a gap of
# 0.5 % of the distance or more at these sizes, so all but stray queries have a proof.
@pytest.mark.parametrize("n,d,k", [(6001, 4, 4), (5857, 10, 8), (6015, 15, 12), (5000, 20, 16), (4001, 31, 20), (3001, 42, 28),
                                   (2500, 64, 31), (20000, 3, 10), (70000, 10, 15)])
def test_matrix_path_answers(n, d, k):
    """General coordinates: nearly every query's list comes from the matrix path, and
    is the one of a scan of all points, bit for bit."""
    x = _mixture(n, d, n)
    idx, d2, scanned = gl.knn_bounded(x, k)
    say(f"knn n={n} d={d} k={k}: {scanned} queries scanned")
    assert scanned <= n // 50
    si, sd, every = gl.knn_bounded(x, k, temp_bytes=1)
    assert every == n
    assert torch.equal(idx, si) and torch.equal(d2, sd)
    gi, gd = gl.knn(x, k)
    assert torch.equal(idx, gi) and torch.equal(d2, gd)


def test_ties_are_scanned():
    """Copies at the k-th place: their queries, at least, have no proof (a point whose k-th
    neighbour is a copy has none either)."""
    n, tied = 9000, 6000
    _, _, scanned = gl.knn_bounded(_points(n, 5, tied, 3), 12)
    say(f"{scanned} of {n} queries scanned, {tied} points in copies")
    assert tied <= scanned <= n


def test_bounded_arguments():
    x = _mixture(500, 3, 1)
    with pytest.raises(gl.GLError):
        gl.knn_bounded(x, 0)
    with pytest.raises(gl.GLError):
        gl.knn_bounded(x.double(), 3)
    assert gl.knn_bounded(x, 3)[2] == 500  # few points: scanned
    assert gl.knn_bounded(_mixture(1000, 80, 2), 5)[2] <= 50  # wide: rescans of the certificate


# wide features: one block of 256 points (every fourth point per segment), several, and a
# full round of 64 query blocks with a few left over; both list lengths
@pytest.mark.parametrize("n,d,k", [(300, 65, 5), (700, 80, 13), (5000, 100, 10), (16500, 70, 12), (17500, 96, 20)])
def test_wide_in_passes(n, d, k):
    """Where the candidate lists of all queries cannot be had, the query blocks are taken
    in passes: the same lists, down to one block per pass, and refused below that."""
    x = _mixture(n, d, n + d)
    idx, d2, _ = gl.knn_bounded(x, k)
    np_, dp = (n + 255) // 256 * 256, (d + 31) // 32 * 32
    fixed = np_ * (2 * dp + 4) + 8 * n + d * (4 + 8 * 256) + 8 * 256  # operands, norms, list of rescans, means, alignment
    per = 64 * (8 if k <= 12 else 12) * 8  # bytes of lists per query, at most
    for blocks in (64, 37, 8, 3, 1):
        bi, bd, _ = gl.knn_bounded(x, k, temp_bytes=fixed + blocks * 256 * per)
        assert torch.equal(bi, idx) and torch.equal(bd, d2), blocks
    if n >= 5000:  # about what a call took with 64 candidates of 4 bytes per query
        bi, bd, _ = gl.knn_bounded(x, k, temp_bytes=n * (2 * dp + 300))
        assert torch.equal(bi, idx) and torch.equal(bd, d2)
    with pytest.raises(gl.GLError, match="memory"):
        gl.knn_bounded(x, k, temp_bytes=2 * np_ * dp)
