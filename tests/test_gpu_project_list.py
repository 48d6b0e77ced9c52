"""The projection's list of (range, view) pairs over more views than one word of
its view mask holds: 130 views of a last mask of two bits, 274 ranges of surfels
(more pairs than the list starts at), a ragged last range, and a map whose
surfels, by their order, leave most ranges outside most views.

Records, rectangles and tile counts equal the oracle's bit for bit, and the batch
renders bitwise the images that each group of views renders by itself without
the list."""
import dataclasses
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2405_14342_amd import binding as B
from paper_2405_14342_amd import synth
from paper_2405_14342_amd.pipeline import TrainState

pytestmark = pytest.mark.gpu

V, N = 130, 70001
GROUP = 26


def _cameras(rng):
    cams = []
    for k in range(V):
        w, h = int(rng.integers(1, 90)), int(rng.integers(1, 60))
        pos = np.array([rng.uniform(0, 80), rng.uniform(-3, 3), rng.uniform(0.5, 4)])
        if k % 5 == 0:
            cam = synth.ortho_bev_camera(pos[:2], 8.0, w, h, m_per_px=float(rng.uniform(0.01, 0.2)))
        else:
            cam = synth.pinhole_camera(pos, rng.uniform(0, 6.28), math.radians(rng.uniform(-90, 20)),
                                       w, h, float(rng.uniform(20, 200)), cull=k % 3 == 0)
        if k % 7 == 3:
            cam.cx, cam.cy = float(rng.uniform(-w, 2 * w)), float(rng.uniform(-h, 2 * h))
        if k % 11 == 5:
            cam.z_near = float(rng.choice([-1.0, 0.0, 1e-3, 2.0]))
        if k in (63, 64, 127, 129):      # the mask's edges see something
            cam = synth.ortho_bev_camera((0.6 * k, 0.0), 8.0, w, h, m_per_px=0.1)
        cams.append(cam)
    return cams


def _scene():
    rng = np.random.default_rng(23)
    x = np.sort(rng.uniform(0, 80, N))          # a range is a stretch of the road
    y, z = rng.uniform(-4, 4, N), rng.normal(0, 0.05, N)
    q = np.concatenate([np.ones((1, N)), rng.normal(0, 0.2, (3, N))])
    s = 10.0 ** rng.uniform(-2.5, -0.5, (2, N))
    s[:, ::997] = 5.0
    return synth.custom_scene(x, y, z, q, s, np.full(N, 0.3), rng.uniform(0, 1, (3, N)),
                              rng.normal(0, 1, (1, N)), _cameras(rng), targets=[])


def _render(sc, cams):
    st = TrainState(dataclasses.replace(sc, cams=cams), opts=B.make_opts())
    ws, _ = st.project_and_sort(st.cams, "cap_batch", "_ws_batch")
    rec = st.rg.debug_records(ws, len(cams), N)
    st.rg.render_fwd(st.surfels(), ws, st.out)
    torch.cuda.synchronize()
    return rec, st.out.cpu().numpy().ravel()


def test_more_views_than_a_mask_word():
    nb = (N + 255) // 256
    assert V * nb > 32768 >= GROUP * nb         # kProjListMin: listed, and direct by groups
    sc = _scene()
    cams = sc.cams
    (rec, rect, cnt), img = _render(sc, cams)
    prm = oracle.Params.from_scene(sc)
    o = oracle.Opts()
    seen = np.zeros(V, np.int64)
    for v, cam in enumerate(cams):
        _, rrec, rrect = oracle.contract(prm, cam, o)
        _, ids, _ = oracle.tile_lists(prm, cam, o)
        ref = np.bincount(ids, minlength=N)
        np.testing.assert_array_equal(cnt[v], ref, err_msg=f"camera {v}")
        on = ref > 0
        np.testing.assert_array_equal(rec[v][on], rrec[on])
        np.testing.assert_array_equal(rect[v][on], rrect[on])
        seen[v] = on.sum()
    assert (seen > 0).sum() > 60 and all(seen[v] > 0 for v in (63, 64, 127, 129))
    parts = [_render(sc, cams[k:k + GROUP])[1] for k in range(0, V, GROUP)]
    np.testing.assert_array_equal(img.view(np.uint32), np.concatenate(parts).view(np.uint32))
