"""More runs to merge than the merge has blocks: 1140 tiles whose lists hold the
same 1100 or 2100 surfels each (2 and 3 runs), in ascending t_z, ties by id."""
import numpy as np
import pytest
import torch

from paper_2405_14342_amd import synth
from paper_2405_14342_amd.pipeline import TrainState

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1100, 2100])
def test_many_lists_of_several_runs(n):
    rng = np.random.default_rng(n)
    z = np.round(rng.uniform(0.0, 4.0, n), 2)                # ties
    q = np.tile(np.array([[1.0], [0.0], [0.0], [0.0]]), (1, n))
    cam = synth.ortho_bev_camera((0.0, 0.0), 10.0, 608, 480, m_per_px=0.01)
    # every footprint covers the whole image
    sc = synth.custom_scene(*rng.uniform(-0.1, 0.1, (2, n)), z, q, np.full((2, n), 3.0),
                            np.full(n, 0.5), np.zeros((3, n)), np.zeros((1, n)), [cam], targets=[])
    st = TrainState(sc)
    ws, pairs = st.project_and_sort(st.cams, "cap_batch", "_ws_batch")
    tiles = 38 * 30
    assert pairs == n * tiles
    _, ids, _, ranges = st.rg.debug_pairs(ws, pairs, tiles)
    rec, _, _ = st.rg.debug_records(ws, 1, n)
    order = np.lexsort((np.arange(n), rec[0, :, 7]))
    assert (ranges[:, 1] - ranges[:, 0] == n).all()
    for a, b in ranges:
        np.testing.assert_array_equal(ids[a:b], order)
    torch.cuda.synchronize()
