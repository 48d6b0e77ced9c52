"""Paths that a batch's size chooses: the tile layout in one pass (up to 4096
tiles) or three launches, the forward's walk in groups of four entries with a
remainder, with and without the semantic sums, and the overflow flag between
projection and binning."""
import math

import numpy as np
import pytest
import torch

from paper_2405_14342_amd import binding as B
from paper_2405_14342_amd import synth
from paper_2405_14342_amd.pipeline import TrainState

pytestmark = pytest.mark.gpu


def _state(n, w, h, C=2, seed=5):
    rng = np.random.default_rng(seed)
    cam = synth.ortho_bev_camera(np.zeros(2), 10.0, w, h, m_per_px=0.01)
    cam.cx, cam.cy = 512.0, 512.0                # the same pixels whatever the width
    xy = rng.uniform(-5.0, 5.0, (2, n))
    s = 10.0 ** rng.uniform(-1.7, -0.7, (2, n))
    q = rng.normal(0, 0.1, (4, n))
    q[0] = 1.0
    sc = synth.custom_scene(*xy, rng.normal(0, 0.1, n), q, s, rng.uniform(0.05, 0.6, n),
                            rng.uniform(0, 1, (3, n)), rng.normal(0, 1, (C, n)), [cam], targets=[])
    return TrainState(sc, opts=B.make_opts(tile_w=16, tile_h=16))


def _render(st, w, h, C=2, channels=None):
    ws, _ = st.project_and_sort(st.cams, "cap_batch", "_ws_batch")
    out = torch.zeros((5 + C, h, w), device="cuda")
    st.rg.render_fwd(st.surfels(), ws, out, channels=channels)
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("w", [1008, 1024, 1040, 2064])
def test_layout_does_not_change_a_tile(w):
    """4032 and 4096 tiles are laid out in one pass, 4160 and 8256 in three
    launches: the shared columns are the same bits."""
    ref = _render(_state(6000, 1024, 1024), 1024, 1024)
    assert float(ref[4 + 2].max()) > 0.5
    out = _render(_state(6000, w, 1024), w, 1024)
    k = min(w, 1024) - 64                        # footprints cut by the border differ in no bit
    assert torch.equal(out[:, :, :k], ref[:, :, :k])


@pytest.mark.parametrize("n", [1, 3, 4, 5, 63, 64, 65, 130, 700])
def test_channel_sets_are_the_same_bits(n):
    """Any selection of planes equals those planes of the full image, for lists
    around the walk's group of 4 and batch of 64."""
    C, w, h = 2, 48, 32
    st = _state(n, w, h, C, seed=n)
    st_c = _state(n, w, h, C, seed=n)
    ref = _render(st, w, h, C)
    rows = {B.CH_RGB: slice(0, 3), B.CH_SEM: slice(3, 3 + C), B.CH_D: slice(3 + C, 4 + C),
            B.CH_A: slice(4 + C, 5 + C)}
    for mask in range(1, 16):
        bits = [b for k, b in enumerate(rows) if mask >> k & 1]
        out = _render(st_c, w, h, C, channels=sum(bits))
        for b in bits:
            assert torch.equal(out[rows[b]], ref[rows[b]]), (n, mask)


def test_overflow_is_known_before_binning():
    st = _state(2000, 256, 256)
    surf = st.surfels()
    for cap, full in ((1 << 20, False), (64, True)):
        ws = torch.empty(B.workspace_size(surf, st.cams, st.opts, cap), dtype=torch.uint8,
                         device="cuda")
        st.rg.project(surf, st.cams, st.opts, ws, cap)
        n, overflow = st.rg.pair_count(ws)
        assert bool(overflow) == full and n > 64


@pytest.mark.parametrize("chunk", [64, 40, 128])
def test_export_restarts_after_an_overflow(chunk):
    """Chunk counts are read a few chunks at a time: an export that overflows
    and is repeated with the capacity it reports gives the same bits and the
    same largest count as one with room from the start."""
    st = _state(3000, 64, 64)
    args = (-0.9, -0.6, 180, 120, 0.01, chunk, 10.0, B.CH_RGB | B.CH_A | B.CH_ELEV)
    out = [torch.zeros((5, 120, 180), device="cuda") for _ in range(2)]
    n0 = st.rg.bev_export(st.surfels(), st.opts, *args, out[0])
    n1 = st.rg.bev_export(st.surfels(), st.opts, *args, out[1], pair_capacity=16)
    torch.cuda.synchronize()
    assert n0 == n1 > 16
    assert float(out[0][3].max()) > 0.3
    assert torch.equal(out[0].nan_to_num(-1.0), out[1].nan_to_num(-1.0))
