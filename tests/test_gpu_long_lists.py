"""Depth order of one tile's list at the lengths where its sort changes form:
one wave up to 511 entries, one block up to 1024, runs of 1024 merged beyond
that.  The order is ascending t_z (binary32), ties by surfel id."""
import numpy as np
import pytest
import torch

from paper_2405_14342_amd import binding as B
from paper_2405_14342_amd import synth
from paper_2405_14342_amd.pipeline import TrainState

pytestmark = pytest.mark.gpu

LENGTHS = [1, 63, 64, 511, 512, 1023, 1024, 1025, 2047, 2048, 2049, 4096, 6145, 16383, 16384, 40000]


@pytest.mark.parametrize("depths", ["distinct", "few", "equal"])
@pytest.mark.parametrize("n", LENGTHS)
def test_one_list(n, depths):
    rng = np.random.default_rng(n)
    # every surfel inside the only tile of a 16 x 16 top-down image
    x, y = rng.uniform(0.3, 0.5, (2, n))
    z = {"distinct": rng.uniform(0.0, 4.0, n), "few": np.round(rng.uniform(0.0, 4.0, n)),
         "equal": np.zeros(n)}[depths]
    q = np.tile(np.array([[1.0], [0.0], [0.0], [0.0]]), (1, n))
    cam = synth.ortho_bev_camera((0.4, 0.4), 10.0, 16, 16, m_per_px=0.05)
    sc = synth.custom_scene(x, y, z, q, np.full((2, n), 0.02), np.full(n, 0.5),
                            np.zeros((3, n)), np.zeros((1, n)), [cam], targets=[])
    st = TrainState(sc)
    ws, pairs = st.project_and_sort(st.cams, "cap_batch", "_ws_batch")
    assert pairs == n
    _, ids, _, ranges = st.rg.debug_pairs(ws, n, 1)
    assert tuple(ranges[0]) == (0, n)
    rec, _, _ = st.rg.debug_records(ws, 1, n)
    tz = rec[0, :, 7]
    np.testing.assert_array_equal(ids[:n], np.lexsort((np.arange(n), tz)))
    torch.cuda.synchronize()
