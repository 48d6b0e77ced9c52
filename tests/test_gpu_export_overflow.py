"""An export whose capacity a chunk exceeds: ROGS_ECAPACITY with the largest
count so far, the chunks before it complete, and neither that chunk nor a later
one written."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2405_14342_amd import binding as B
from paper_2405_14342_amd import synth
from paper_2405_14342_amd.pipeline import TrainState

pytestmark = pytest.mark.gpu
W, H, CHUNK, M, HEIGHT = 200, 150, 48, 0.02, 10.0
CHANNELS = B.CH_RGB | B.CH_A | B.CH_ELEV


def _state():
    rng = np.random.default_rng(4)
    n = 4000
    # denser towards the chunks that come last
    x, y = W * M * np.sqrt(rng.uniform(0, 1, n)), H * M * (1.0 - np.sqrt(rng.uniform(0, 1, n)))
    q = np.concatenate([np.ones((1, n)), rng.normal(0, 0.1, (3, n))])
    cam = synth.ortho_bev_camera((1.0, 1.0), HEIGHT, 64, 64, m_per_px=M)
    sc = synth.custom_scene(x, y, rng.normal(0, 0.1, n), q, 10.0 ** rng.uniform(-2, -1.3, (2, n)),
                            rng.uniform(0.1, 0.7, n), rng.uniform(0, 1, (3, n)),
                            rng.normal(0, 1, (2, n)), [cam], targets=[])
    return TrainState(sc)


def _export(st, out, cap):
    L, surf, size, worst = B.load_library(), st.surfels(), ctypes.c_size_t(0), ctypes.c_int64(-1)
    assert L.rogs_bev_workspace_size(ctypes.byref(surf), CHUNK, ctypes.byref(st.opts), cap,
                                     ctypes.byref(size)) == B.OK
    ws = torch.empty(size.value, dtype=torch.uint8, device="cuda")
    r = L.rogs_bev_export(st.rg.h, ctypes.byref(surf), ctypes.byref(st.opts), 0.0, 0.0, W, H, M,
                          CHUNK, HEIGHT, CHANNELS, B.ptr(out), B.ptr(ws), size.value, cap,
                          ctypes.byref(worst), B._stream(None))
    torch.cuda.synchronize()
    return r, worst.value


def _chunks():
    return [(oy, ox) for oy in range(0, H, CHUNK) for ox in range(0, W, CHUNK)]


@pytest.mark.parametrize("at", [0, 1, 2, 3, -1])
def test_an_overflowing_chunk_is_not_written(at):
    st = _state()
    counts = []
    for oy, ox in _chunks():
        cam = B.bev_camera(0.0, 0.0, W, H, M, ox, oy, min(CHUNK, W - ox), min(CHUNK, H - oy), HEIGHT)
        counts.append(st.project_and_sort([cam], "cap_view", "_ws_view")[1])
    planes = B.channel_planes(CHANNELS, 2)
    full = torch.full((planes, H, W), -7.0, device="cuda")
    assert _export(st, full, max(counts)) == (B.OK, max(counts))
    # chunks whose count passes all of those before them
    peaks = [k for k in range(len(counts)) if counts[k] > max(counts[:k], default=0)]
    assert len(peaks) >= 5
    first = peaks[at]
    out = torch.full_like(full, -7.0)
    assert _export(st, out, counts[first] - 1) == (B.ECAPACITY, counts[first])
    for k, (oy, ox) in enumerate(_chunks()):
        a, b = (t[:, oy:oy + CHUNK, ox:ox + CHUNK] for t in (out, full))
        if k < first:
            assert torch.equal(a.nan_to_num(-1.0), b.nan_to_num(-1.0)), k
        else:
            assert (a == -7.0).all(), k


def test_no_backward_after_an_export():
    """rogs_render_bwd needs a rogs_render_fwd of every plane: the images of an
    export lie in the stitched image, not in the batch's layout."""
    st = _state()
    L, surf, size, worst = B.load_library(), st.surfels(), ctypes.c_size_t(0), ctypes.c_int64(0)
    cap = 1 << 18
    assert L.rogs_bev_workspace_size(ctypes.byref(surf), 64, ctypes.byref(st.opts), cap,
                                     ctypes.byref(size)) == B.OK
    ws = torch.empty(size.value, dtype=torch.uint8, device="cuda")
    out = torch.empty((B.channel_planes(B.CH_ALL, 2), 64, 64), device="cuda")
    assert L.rogs_bev_export(st.rg.h, ctypes.byref(surf), ctypes.byref(st.opts), 0.0, 0.0, 64, 64, M,
                             64, HEIGHT, B.CH_ALL, B.ptr(out), B.ptr(ws), size.value, cap,
                             ctypes.byref(worst), B._stream(None)) == B.OK
    G = torch.zeros_like(out)
    with pytest.raises(B.RogsError, match="ESTATE"):
        st.rg.render_bwd(surf, ws, out, G, st.grads)
