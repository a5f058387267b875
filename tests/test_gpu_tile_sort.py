"""The tile sort at the lengths where its paths change: depth order with ties by index, bit-exact
against numpy, for lists of one wave's run, several runs (whole, partial, an odd number), the
largest of each kernel and one more, and for sessions with more binning chunks than the gather
keeps in LDS."""
import numpy as np
import pytest
import torch

from paper_2510_06644_amd import rtgs, synth
from tests.gpu_util import eye_view

pytestmark = pytest.mark.gpu


def _lists(n, visible, seed, w=16, h=16):
    """ids and depths of a frame of one tile in which `visible` of n Gaussians are drawn, their
    depths quantised so that many are equal."""
    rng = np.random.default_rng(seed)
    cam = rtgs.Cam(w, h, 20.0, 20.0, w / 2, h / 2)
    z = np.full(n, -1.0, np.float32)
    on = np.sort(rng.choice(n, visible, replace=False))
    z[on] = (1.0 + np.floor(rng.random(visible) * max(visible // 3, 1)) / max(visible // 3, 1) * 4
             ).astype(np.float32)
    means = np.stack([np.zeros(n), np.zeros(n), z], 1).astype(np.float32)
    scene = (means, np.full((n, 3), -4.0, np.float32), np.tile(np.float32([1, 0, 0, 0]), (n, 1)),
             np.full(n, -3.0, np.float32), np.full((n, 3), 0.5, np.float32))
    R = rtgs.Renderer(0, pairs_per_gaussian=2.0)
    st = R.forward(tuple(torch.from_numpy(a).cuda() for a in scene),
                   torch.from_numpy(eye_view()).cuda(), cam)
    return st.stage()["ids"], on[np.lexsort((on, z[on]))]


@pytest.mark.parametrize("n", [1, 2, 63, 255, 256, 257, 511, 513, 769, 1023, 1024, 1025, 1535, 2047,
                               2048, 2049, 3000, 4096, 4097, 8191, 8192, 8193, 20000])
def test_list_lengths(n):
    ids, want = _lists(n, n, n)
    assert np.array_equal(ids, want)


@pytest.mark.parametrize("visible", [700, 1800, 2500])
def test_more_chunks_than_the_run_table(visible):
    ids, want = _lists(1_050_000, visible, visible)
    assert np.array_equal(ids, want)
