"""Thin, tilted footprints in tiles of one, two and four waves against the
oracle's lists and records: a list entry that a wave leaves out although it
reaches one of the wave's pixels shows in the image.

The reference composites in binary64 with the oracle's binary32 test value q
(oracle.q32) both as the test and in the weight, as the library does: on a thin
conic the binary32 value itself is up to 1e-4 from the binary64 one.

Tolerance per pixel with n contributing entries of opacity a <= 0.6, in units of
2^-23: a weight's factors (q's scaling, exp2, a) are off by at most 4; a factor
1 - a of the transmittance by 4 a / (1 - a) + 1/2 <= 6.5; a product and a sum
each round once more.  So no entry's share is off by more than 7 n + 8 of it,
and the shares add up to at most the largest feature; pixels may stop one entry
apart, which leaves t_eps of it."""
import numpy as np
import pytest
import torch

import oracle
from paper_2405_14342_amd import binding as B
from paper_2405_14342_amd.pipeline import TrainState
from test_gpu_parts import thin_scene

pytestmark = pytest.mark.gpu


def _composite(prm, cam, o):
    """rgb, semantics and alpha planes, and the contributing entries per pixel."""
    _, rec, _ = oracle.contract(prm, cam, o)
    _, ids, ranges = oracle.tile_lists(prm, cam, o)
    feat = np.concatenate([prm.rgb, prm.sem]).astype(np.float64)
    out = np.zeros((len(feat) + 1, cam.h, cam.w))
    count = np.zeros((cam.h, cam.w), np.int64)
    tx = (cam.w + o.tile_w - 1) // o.tile_w
    for t, (a, b) in enumerate(ranges):
        if a == b:
            continue
        y0, x0 = t // tx * o.tile_h, t % tx * o.tile_w
        y1, x1 = min(y0 + o.tile_h, cam.h), min(x0 + o.tile_w, cam.w)
        py, px = (v.ravel() for v in np.mgrid[y0:y1, x0:x1])
        lst = ids[a:b]
        q = oracle.q32(rec[lst], px, py)
        T = np.ones(px.size)
        acc = np.zeros((len(feat), px.size))
        n = np.zeros(px.size, np.int64)
        for k, i in enumerate(lst):
            on = (q[k] <= np.float32(o.q_cut)) & (T >= o.t_eps)
            w = np.where(on, float(prm.alpha[i]) * np.exp(-0.5 * q[k].astype(np.float64)), 0.0)
            acc += feat[:, i:i + 1] * (w * T)
            T *= 1.0 - w
            n += on
        out[:-1, y0:y1, x0:x1] = acc.reshape(len(feat), y1 - y0, x1 - x0)
        out[-1, y0:y1, x0:x1] = (1.0 - T).reshape(y1 - y0, x1 - x0)
        count[y0:y1, x0:x1] = n.reshape(y1 - y0, x1 - x0)
    return out, count


@pytest.mark.parametrize("tile", [(16, 4), (16, 8), (8, 16), (64, 2), (16, 16), (64, 4), (8, 32)])
def test_thin_footprints(tile):
    C = 3
    sc = thin_scene(C)
    st = TrainState(sc, opts=B.make_opts(tile_w=tile[0], tile_h=tile[1]))
    ws, _ = st.project_and_sort(st.cams, "cap_batch", "_ws_batch")
    st.rg.render_fwd(st.surfels(), ws, st.out)
    torch.cuda.synchronize()
    img = st.out.cpu().numpy().ravel().astype(np.float64)
    prm = oracle.Params.from_scene(sc)
    o = oracle.Opts(*tile)
    off = 0
    for v, cam in enumerate(sc.cams):
        got = img[off:off + (5 + C) * cam.w * cam.h].reshape(5 + C, cam.h, cam.w)
        off += got.size
        ref, n = _composite(prm, cam, o)
        fmax = np.concatenate([np.abs(prm.rgb).max(1), np.abs(prm.sem).max(1), [1.0]])
        tol = fmax[:, None, None] * ((7 * n + 8) * 2.0 ** -23 + 2 * o.t_eps)
        err = np.abs(got[[*range(3 + C), 4 + C]] - ref)
        assert n.max() > 8 and (n == 0).any()
        assert (err <= tol).all(), (v, tile, (err / tol).max())
