"""gl_knn_graph on both sides of the choice between rows and one sort: the smallest
graphs, whose weight array has just the room for the rows' lengths, hubs, and
lists that all name the same few points."""

import numpy as np
import pytest
import torch

import paper_2303_14495_amd as gl
from oracle import knn_oracle
from tests.gpu_helpers import DEV, say

pytestmark = pytest.mark.gpu


def _lists(n, k, kind):
    """(idx, d2): distinct neighbours per row; d2 a symmetric function of the pair."""
    rng = np.random.default_rng(n * 31 + k)
    i = np.arange(n)
    idx = np.empty((n, k), np.int32)
    pool = {"few": max(k + 1, n // 12), "hub": n, "any": n}[kind]
    for r in range(n):
        pick = rng.choice(pool, k + 1, replace=False)
        idx[r] = pick[pick != r][:k]
        if kind == "hub" and r != 3 and 3 not in idx[r]:
            idx[r, 0] = 3
    lo, hi = np.minimum(i[:, None], idx).astype(np.int64), np.maximum(i[:, None], idx).astype(np.int64)
    return idx, (0.25 + (lo * 29 + hi * 13) % 101 / 64.0).astype(np.float32)


# rows longer than 4096 entries, and more than one in 16 of over 64, go to the sort, as do
# lists of 25 and more; its keys have as many bits as n - 1, twice: both sides of powers of two
@pytest.mark.parametrize("n,k,kind", [(2, 1, "any"), (3, 1, "any"), (3, 2, "any"), (5, 4, "any"), (65, 24, "any"), (66, 25, "any"),
                                      (4095, 2, "hub"), (4300, 3, "hub"), (1300, 10, "few"), (700, 24, "few"), (257, 7, "few"),
                                      (26, 25, "any"), (32, 25, "any"), (33, 25, "any"), (64, 30, "any"), (65, 30, "any"),
                                      (128, 100, "any"), (129, 26, "few"), (1024, 30, "any"), (1025, 30, "any")])
def test_against_the_oracle(n, k, kind):
    idx, d2 = _lists(n, k, kind)
    rp, col, w = (t.cpu().numpy() for t in gl.knn_graph(torch.from_numpy(idx).to(DEV), torch.from_numpy(d2).to(DEV), k))
    orp, ocol, ow = knn_oracle.graph_from_knn(n, idx, d2.astype(np.float64), k)
    say(f"knn graph {kind} n={n} k={k}: longest row {int(np.diff(orp).max())}")
    assert rp.tolist() == orp.tolist() and col.tolist() == ocol.tolist()
    assert np.all(np.abs(w - ow) <= 4 * np.spacing(ow))  # one division and exponential on both sides


@pytest.mark.parametrize("kind", ["any", "hub"])
def test_defects_in_either(kind):
    idx, d2 = _lists(4300, 3, kind)
    for what in ("range", "self", "negative", "nan"):
        bi, bd = idx.copy(), d2.copy()
        if what == "range":
            bi[4299, 2] = 4300
        elif what == "self":
            bi[17, 0] = 17
        elif what == "negative":
            bd[4000, 1] = -1.0
        else:
            bd[0, 0] = np.nan
        with pytest.raises(gl.GLError):
            gl.knn_graph(torch.from_numpy(bi).to(DEV), torch.from_numpy(bd).to(DEV), 3)


# 2^21 list entries and more: four times the entries per workgroup of the count
@pytest.mark.parametrize("n,k,hub", [(209715, 10, True), (209720, 10, True), (209720, 10, False), (110000, 20, False)])
def test_large_structure(n, k, hub):
    """Row offsets and columns of the union of random lists, with a point in all of them or none."""
    g = torch.Generator(device=DEV)
    g.manual_seed(n + k)
    i = torch.arange(n, device=DEV)
    step = torch.randint(1, n // k, (n, k), generator=g, device=DEV) + torch.arange(k, device=DEV) * (n // k)
    idx = (i[:, None] + step) % n
    if hub:
        idx[:, 0] = torch.where((idx[:, 1:] == 7).any(1) | (i == 7), idx[:, 0], 7)
    d2 = torch.sort(torch.rand(n, k, generator=g, device=DEV), 1).values + 0.1
    rp, col, w = gl.knn_graph(idx.to(torch.int32), d2, k)
    a, b = i.repeat_interleave(k), idx.reshape(-1)
    key = torch.unique(torch.cat([a * n + b, b * n + a]))
    want = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    want[1:] = torch.cumsum(torch.bincount(key // n, minlength=n), 0)
    say(f"knn graph n={n} k={k}: longest row {int((want[1:] - want[:-1]).max())}")
    assert torch.equal(rp, want) and torch.equal(col.to(torch.int64), key % n)
    assert bool((w > 0).all())
