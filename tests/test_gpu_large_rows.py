"""Operator construction at row counts whose 16 lanes per row are more threads
than one dimension of a launch holds."""

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
