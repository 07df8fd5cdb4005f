"""Row and point counts whose lanes are more than one row of a folded grid, or more
than one dimension of a launch, holds."""

import pytest
import torch

import paper_2303_14495_amd as gl
from tests.gpu_helpers import DEV, say

pytestmark = pytest.mark.gpu


# 2^28 rows have 2^32 lanes
@pytest.mark.parametrize("n", [2**28, 2**28 + 2 * 16384 + 2])
def test_pairs(n):
    """Rows i and i ^ 1 joined by an edge: L_s x = x_i - x_(i ^ 1)."""
    if torch.cuda.mem_get_info()[0] < 40e9:
        pytest.skip("needs 40 GB of device memory")
    i = torch.arange(n + 1, device=DEV)
    op = gl.Operator(i, (i[:-1] ^ 1).to(torch.int32), torch.full((n,), 0.5, dtype=torch.float32, device=DEV), store_w="f32")
    x = (i[:-1] % 1021).to(torch.float32).unsqueeze(1)
    y = op.laplacian_apply(x)
    pairs = x.view(-1, 2)
    want = torch.stack([pairs[:, 0] - pairs[:, 1], pairs[:, 1] - pairs[:, 0]], 1).view(-1, 1)
    # the weight is 0.5 / (sqrt(0.5) sqrt(0.5)) in double, rounded once: 1 or 1 - 2^-24
    worst = float((y - want).abs().max())
    say(f"pairs n={n}: max error {worst:.1e}")
    assert worst <= 1021 * 2.0**-23
    op.close()
    # a defect in the last row is found
    w = torch.full((n,), 0.5, dtype=torch.float32, device=DEV)
    w[n - 1] = 0.25
    with pytest.raises(gl.GLError, match="symmetric"):
        gl.Operator(i, (i[:-1] ^ 1).to(torch.int32), w, store_w="f32")


# a wavefront per query fills one row of the folded grid at 4 * 65 536 points, 26
# operand vectors per point of 64 coordinates at 645 277
@pytest.mark.parametrize("n,d,span", [(300_001, 3, 200), (646_000, 64, 200)])
def test_knn_folded(n, d, span):
    """Integer coordinates, whose distances are exact: lists with ties to the lower index."""
    k = 10
    g = torch.Generator(device=DEV)
    g.manual_seed(n)
    x = torch.randint(0, span, (n, d), generator=g, device=DEV).float()
    idx, d2 = gl.knn(x, k)
    edge = 4 * 65536
    rows = [0, 1, edge - 2, edge - 1, edge, edge + 1, 2 * edge, 2 * edge + 1, n - 33, n - 2, n - 1]
    rows += torch.randint(0, n, (20,), generator=g, device=DEV).tolist()
    for q in (r for r in rows if r < n):
        dist = ((x - x[q]) ** 2).sum(1).to(torch.int64)  # whole numbers below 2^24
        key = dist * n + torch.arange(n, device=DEV)
        key[q] = 2**62
        best = torch.sort(torch.topk(key, k, largest=False).values).values
        assert torch.equal(idx[q].to(torch.int64), best % n), q
        assert torch.equal(d2[q].to(torch.int64), best // n), q
    say(f"knn n={n} d={d}: {len(rows)} rows")


def test_window_of_a_tall_image():
    """One column of 2^25 + 5 pixels of one colour: its two strips are 2^32 threads when the
    weights are stored.  Every weight is 1, degrees 1 at the ends and 2 inside."""
    if torch.cuda.mem_get_info()[0] < 100e9:
        pytest.skip("needs 100 GB of device memory")
    n = 2**25 + 5
    op = gl.Operator.window(torch.full((n, 1, 1), 0.5, device=DEV), window_radius=1, patch_radius=1, sigma=1.0, store_w="f32")
    x = (torch.arange(n, device=DEV) % 509).to(torch.float32).unsqueeze(1)
    y = op.laplacian_apply(x)[:, 0]
    r = torch.full((n,), 2.0, device=DEV)
    r[0] = r[-1] = 1.0
    v = x[:, 0]
    edge = 1.0 / (r[1:] * r[:-1]).sqrt()
    want = v.clone()
    want[1:] -= edge * v[:-1]
    want[:-1] -= edge * v[1:]
    worst = float((y - want).abs().max())
    say(f"window of {n} x 1: max error {worst:.1e}")
    assert worst <= 4 * 509 * 2.0**-23  # two products of values below 509 and weights of at most 1
    op.close()
