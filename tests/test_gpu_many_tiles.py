"""A batch with more tiles than one grid holds at four waves each (2^24 blocks of
256 threads are 2^32): 1025 views of 16384 x 1 in tiles of 1 x 256.  Every tile
is composited and differentiated: images and gradients are those of the same
views one at a time, and the fused step is the batched step."""
import numpy as np
import pytest
import torch

from paper_2405_14342_amd import binding as B
from paper_2405_14342_amd import synth
from paper_2405_14342_amd.pipeline import TrainState

pytestmark = pytest.mark.gpu
VIEWS, W = 1025, 16384


def _scene():
    rng = np.random.default_rng(8)
    n = 40
    x = np.linspace(0.0, W * 0.01, n)
    q = np.concatenate([np.ones((1, n)), np.zeros((3, n))])
    cams = [synth.ortho_bev_camera((0.5 * W * 0.01 + 0.02 * k, 0.0), 10.0, W, 1, m_per_px=0.01)
            for k in range(VIEWS)]
    return synth.custom_scene(x, rng.normal(0, 0.01, n), rng.normal(0, 0.1, n), q,
                              10.0 ** rng.uniform(-1.5, -0.8, (2, n)), rng.uniform(0.2, 0.7, n),
                              rng.uniform(0.2, 1, (3, n)), rng.normal(0, 1, (1, n)), cams, targets=[])


def _state():
    st = TrainState(_scene(), opts=B.make_opts(tile_w=1, tile_h=256))
    gen = torch.Generator("cuda").manual_seed(3)
    st.G.copy_(torch.randn(st.G.numel(), generator=gen, device="cuda"))
    npix = VIEWS * W
    assert npix > 1 << 24                       # one tile per pixel
    st.tgt_rgb = torch.rand(3 * npix, generator=gen, device="cuda")
    st.tgt_label = torch.zeros(npix, dtype=torch.uint8, device="cuda")
    st.tgt_mask = torch.ones(npix, dtype=torch.uint8, device="cuda")
    return st


def test_images_and_gradients():
    st = _state()
    surf = st.surfels()
    ws, _ = st.project_and_sort(st.cams, "cap_batch", "_ws_batch")
    st.out.fill_(-7.0)
    st.rg.render_fwd(surf, ws, st.out)
    st.rg.render_bwd(surf, ws, st.out, st.G, st.grads)
    out, acc = torch.full_like(st.out, -7.0), torch.zeros_like(st.grads)
    per = (5 + st.C) * W
    for v in range(VIEWS):
        ws, _ = st.project_and_sort(st.cams[v:v + 1], "cap_view", "_ws_view")
        o = out[v * per:(v + 1) * per]
        st.rg.render_fwd(surf, ws, o)
        st.rg.render_bwd(surf, ws, o, st.G[v * per:(v + 1) * per], acc, B.ACCUMULATE if v else 0)
    torch.cuda.synchronize()
    assert torch.equal(out, st.out) and float(out.max()) > 0.5
    # the views' sums are added in the same order in both
    assert torch.equal(acc, st.grads) and float(acc.abs().max()) > 0


def test_fused_step():
    a, b = _state(), _state()
    a.step_batched(total_steps=5)
    b.step_fused(total_steps=5, grads_out=True)
    torch.cuda.synchronize()
    for k in ("grads", "params", "m", "v"):
        assert torch.equal(getattr(a, k), getattr(b, k)), k
    # a view's loss is a sum of the same positive terms at most 80 adds deep in
    # both, and the views are added in the same order
    loss = a.loss.item()
    assert loss > 0 and abs(b.fused_status()["loss"] - loss) <= 200 * 2.0 ** -24 * loss


def test_mask_counts_of_mixed_views():
    """One view of 16384 x 8193 and 1029 of 8 x 8: the fused step's mask chunks,
    counted per view by the largest view's number, are more blocks than one grid
    holds.  Each view's loss is divided by its own mask count: the fused step is
    the batched step."""
    rng = np.random.default_rng(12)
    n = 8300                                   # 33 ranges x 1030 views: pairs are listed
    cams = [synth.ortho_bev_camera((20.0, 20.0), 10.0, 16384, 8193, m_per_px=0.0025)]
    cams += [synth.ortho_bev_camera(rng.uniform(0, 40, 2), 10.0, 8, 8, m_per_px=0.05)
             for _ in range(1029)]
    q = np.concatenate([np.ones((1, n)), np.zeros((3, n))])
    sc = synth.custom_scene(*rng.uniform(0, 40, (2, n)), rng.normal(0, 0.1, n), q,
                            np.full((2, n), 0.02), rng.uniform(0.2, 0.7, n), rng.uniform(0, 1, (3, n)),
                            rng.normal(0, 1, (1, n)), cams, targets=[])

    def state():
        st = TrainState(sc, opts=B.make_opts(tile_w=16, tile_h=16))
        npix = sum(st.npix)
        gen = torch.Generator("cuda").manual_seed(4)
        st.tgt_rgb = torch.rand(3 * npix, generator=gen, device="cuda")
        st.tgt_label = torch.zeros(npix, dtype=torch.uint8, device="cuda")
        st.tgt_mask = (torch.rand(npix, generator=gen, device="cuda") < 0.7).to(torch.uint8)
        return st

    a = state()
    a.step_batched(total_steps=5)
    torch.cuda.synchronize()
    ref = {k: getattr(a, k).clone() for k in ("grads", "params", "m", "v")}
    loss = a.loss.item()
    del a
    torch.cuda.empty_cache()
    b = state()
    b.step_fused(total_steps=5, grads_out=True)
    torch.cuda.synchronize()
    for k, t in ref.items():
        assert torch.equal(t, getattr(b, k)), k
    assert loss > 0 and abs(b.fused_status()["loss"] - loss) <= 200 * 2.0 ** -24 * loss
