"""Places in the workspace that kernels derive from a view's index: the host
checks of tests/layout_driver.cpp (any mix of view sizes, without a GPU), and a
fused step over one large view among hundreds of tiny ones against the batched
step."""
import os
import subprocess

import numpy as np
import pytest
import torch

from paper_2405_14342_amd import binding as B
from paper_2405_14342_amd import synth
from paper_2405_14342_amd.pipeline import TrainState

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
EXE = os.path.join(ROOT, "tests", "_bin", "layout_checks")


def test_layout_holds_any_mix_of_view_sizes():
    assert os.path.exists(EXE), "build the driver first (paper_2405_14342_amd/build.py)"
    r = subprocess.run([EXE], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    assert "layout checks: ok" in r.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("big", [0, 350, 599])
def test_one_large_view_among_tiny_ones(big):
    """600 views, one of 1920 x 1080 and the others 16 x 16, in 16 x 4 tiles: were
    the chunk sums of the tile losses laid out by the largest view's count for
    every view, they would run past their room.  The parameters are the batched
    step's bits.  The loss and dL/d(a, b) sum the same terms in another order:
    at most 40 adds deep over terms whose magnitudes sum to at most 3 / 600 per
    view (the colours and weights are at most 1, the view's scale 1 / 600), so
    they differ by at most 80 2^-24 of that."""
    base = synth.mini_strip(n_along=100, n_across=30, n_sem=3)
    cam = base.cams[0]
    p = -np.asarray(cam.R_cw, np.float64).T @ np.asarray(cam.t_cw, np.float64)
    view = lambda w, h, yaw: synth.pinhole_camera(p, yaw, -0.25, w, h, 0.7 * w)
    cams = [view(1920, 1080, 0.1) if k == big else view(16, 16, 0.01 * k) for k in range(600)]
    sc = synth.custom_scene(base.x, base.y, base.z, base.q, base.s, base.alpha, base.rgb, base.sem,
                            cams)
    opts = lambda: B.make_opts(tile_w=16, tile_h=4)
    a, b = TrainState(sc, opts=opts()), TrainState(sc, opts=opts())
    a.step_batched(total_steps=5)
    b.step_fused(total_steps=5, grads_out=True)
    torch.cuda.synchronize()
    st = b.fused_status()
    assert st["overflow"] == 0 and st["step"] == 1 and st["pairs"] > 1000
    for k in ("grads", "params", "m", "v", "s_act", "alpha_act"):
        assert torch.equal(getattr(a, k), getattr(b, k)), k
    bound = 80 * 2.0 ** -24
    assert abs(st["loss"] - a.loss.item()) <= bound * a.loss.item()
    assert a.d_exp.abs().max().item() > 0
    assert (a.d_exp - b.d_exp).abs().max().item() <= bound * 3.0 / 600
