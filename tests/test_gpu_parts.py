"""Tiles of several waves (128 and 256 pixels), whose waves each leave out the
list entries that cannot reach their own 64 pixels.

- With thin, tilted footprints (axis ratios up to about 60 before projection,
  seen at grazing angles) every shape renders bitwise the same images.
- The fused step equals the batched step plus Adam bit for bit, at every
  staging depth, for one and two blocks of feature columns, and where pixels
  stop early.  With one-wave tiles this compares a forward that leaves nothing
  out (the fused step's) with one that does (the batched step's)."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2405_14342_amd import binding as B
from paper_2405_14342_amd import synth
from paper_2405_14342_amd.pipeline import TrainState

pytestmark = pytest.mark.gpu

SHAPES = [(16, 8), (64, 2), (8, 16), (16, 16), (64, 4), (8, 32)]
SIZES = [(161, 83), (130, 97), (161, 83), (64, 48), (130, 97), (17, 300)]


def thin_scene(n_sem=4):
    sc = synth.mini_strip(n_along=120, n_across=40, n_sem=n_sem, sides=SIZES)
    rng = np.random.default_rng(11)
    s = np.exp(rng.uniform(np.log(0.01), np.log(0.6), (2, sc.n)))
    q = np.concatenate([np.ones((1, sc.n)), rng.normal(0.0, 0.4, (3, sc.n))])
    a = rng.uniform(0.05, 0.6, sc.n)
    return dataclasses.replace(sc, q=q.astype(np.float32), s=s.astype(np.float32),
                               log_s=np.log(s).astype(np.float32), alpha=a.astype(np.float32),
                               logit_a=np.log(a / (1.0 - a)).astype(np.float32))


def test_thin_footprints_every_shape():
    sc = thin_scene()
    first = None
    for tw, th in [(16, 4), *SHAPES]:
        st = TrainState(sc, opts=B.make_opts(tile_w=tw, tile_h=th))
        ws, _ = st.project_and_sort(st.cams, "cap_batch", "_ws_batch")
        st.rg.render_fwd(st.surfels(), ws, st.out)
        torch.cuda.synchronize()
        if first is None:
            first = st
        assert torch.equal(st.out, first.out), (tw, th)


@pytest.mark.parametrize("t_eps", [1e-6, 0.2])
@pytest.mark.parametrize("n_sem,tile,stage", [(4, (16, 4), 32), (4, (64, 1), 16), (8, (8, 8), 64),
                                              (4, (16, 8), 16), (4, (64, 4), 64),
                                              (16, (8, 16), 32), (16, (16, 16), 64)])
def test_fused_equals_batched(n_sem, tile, stage, t_eps):
    sc = thin_scene(n_sem)
    opts = lambda: B.make_opts(tile_w=tile[0], tile_h=tile[1], stage=stage, t_eps=t_eps)
    a, b = TrainState(sc, opts=opts()), TrainState(sc, opts=opts())
    a.step_batched(total_steps=5)
    b.step_fused(total_steps=5, grads_out=True)
    torch.cuda.synchronize()
    assert torch.equal(a.grads, b.grads)
    for k in ("params", "m", "v", "s_act", "alpha_act"):
        assert torch.equal(getattr(a, k), getattr(b, k)), k
