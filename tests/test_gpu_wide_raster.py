"""A raster wider than one grid row of blocks (2^29 cells at 32 cells to a block
of 256 threads): its last columns hold the layout that a raster of those columns
alone gives, the others none.  Spacing and origin are multiples of 1/8 m, so the
cell positions are exact in both."""
import numpy as np
import pytest
import torch

from paper_2405_14342_amd import binding as B

pytestmark = pytest.mark.gpu


def test_last_columns_of_a_wide_raster():
    W, H, cut, h = (1 << 29) + 100, 2, 1 << 29, 0.125
    first = W - 1000                            # the small raster's first column
    rng = np.random.default_rng(6)
    p = np.zeros((30, 12), np.float32)
    p[:, 0] = h * rng.integers(40, 1000, 30)
    p[-1, 0] = h * 999
    p[:, 1] = h * rng.integers(0, 2, 30)
    p[:, 2] = rng.uniform(-1, 1, 30)
    p[:, 3] = p[:, 7] = p[:, 11] = 1.0
    poses = torch.as_tensor(p, device="cuda")
    rg = B.Rogs()
    ref = rg.meshgrid_layout(poses, 0.0, 0.0, h, 1000, H, 12)
    out = rg.meshgrid_layout(poses, -h * first, 0.0, h, W, H, 12)
    torch.cuda.synchronize()
    assert out["n"] == ref["n"] > 500
    assert int((ref["idx"][:, cut - first:] >= 0).sum()) > 10
    for k in ("x", "y", "z", "q", "nbr"):
        assert torch.equal(out[k], ref[k]), k
    assert torch.equal(out["idx"][:, first:], ref["idx"])
    assert all(int((out["idx"][r, :first] != -1).sum()) == 0 for r in range(H))
