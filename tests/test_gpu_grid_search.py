"""The searches over the raster and the point grid at the sizes where their
forms change, against the oracle's brute force, bit for bit: rasters whose rows
do not end on words of 64 cells or blocks of 32 x 8, more poses near a block
than it keeps (512), poses at equal distance, disks that leave the raster; point
grids with empty rows and columns around few cells with points."""
import numpy as np
import pytest
import torch

import oracle
from paper_2405_14342_amd import binding as B

pytestmark = pytest.mark.gpu


def _poses(xy, rng):
    n = len(xy)
    p = np.zeros((n, 12), np.float32)
    p[:, :2] = xy
    p[:, 2] = rng.uniform(-1, 1, n)
    for k in range(n):
        Q, U = np.linalg.qr(np.eye(3) + 0.2 * rng.normal(size=(3, 3)))
        p[k, 3:] = (Q * np.sign(np.diag(U))).reshape(-1)
    return p


@pytest.mark.parametrize("W,H,radius,n", [(1, 1, 0, 1), (63, 9, 3, 5), (64, 8, 200, 2), (65, 17, 12, 40),
                                          (129, 33, 20, 513), (200, 50, 31, 1500), (5, 700, 40, 60)])
def test_layout(W, H, radius, n):
    rng = np.random.default_rng(W * 1000 + n)
    h, x0, y0 = np.float32(0.1), -3.7, 12.3
    # some poses outside the raster, and every pose twice (the lower index wins)
    xy = np.stack([x0 + 0.1 * rng.uniform(-5, W + 5, (n + 1) // 2),
                   y0 + 0.1 * rng.uniform(-5, H + 5, (n + 1) // 2)], 1)
    xy[0] = x0, y0
    poses = _poses(np.concatenate([xy, xy])[:n], rng)
    ref = oracle.meshgrid_layout(poses, x0, y0, h, W, H, radius)
    out = B.Rogs().meshgrid_layout(torch.as_tensor(poses, device="cuda"), x0, y0, h, W, H, radius)
    torch.cuda.synchronize()
    assert out["n"] == ref["x"].size > 0
    for k in ("idx", "x", "y", "z", "nbr"):
        np.testing.assert_array_equal(out[k].cpu().numpy(), ref[k], err_msg=k)
    np.testing.assert_array_equal(out["q"].cpu().numpy(), ref["q"].astype(np.float32))


@pytest.mark.parametrize("n,m", [(1, 1), (300, 2), (2000, 63), (2000, 700), (5000, 20000)])
def test_lidar_corners(n, m):
    """Points in two opposite corners (one on a coarse lattice: ties)."""
    rng = np.random.default_rng(n + m)
    f = lambda a: np.ascontiguousarray(a, np.float32)
    x, y = f(rng.uniform(-40, 60, n)), f(rng.uniform(-7, 13, n))
    px, py = rng.uniform(-40, -38, m), rng.uniform(-7, -6, m)
    px[m // 2:] = 58 + np.round(rng.uniform(0, 2, m - m // 2) * 8) / 8
    py[m // 2:] = 12 + np.round(rng.uniform(0, 1, m - m // 2) * 8) / 8
    px, py = f(px), f(py)
    d = lambda a: torch.as_tensor(a, device="cuda")
    zbar, idx = torch.empty(n, device="cuda"), torch.empty(n, dtype=torch.int32, device="cuda")
    B.Rogs().lidar_targets(d(x), d(y), d(px), d(py), d(f(np.arange(m))), zbar, idx)
    np.testing.assert_array_equal(idx.cpu().numpy(), oracle.lidar_nn(x, y, px, py))
