"""The binning scan's routes by size: chunk counts added in the scan (chunks x
tiles up to 16384) or by a kernel of their own, and tile counts in registers, 4 or
12 a thread.  Tile ranges and lists are bit-exact
against the replay."""
import numpy as np
import pytest
import torch

from oracle import binning
from paper_2510_06644_amd import rtgs, synth
from tests.gpu_util import eye_view, rcam, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,n", [
    (320, 240, 1), (320, 240, 20_000), (1024, 1024, 4096), (1024, 1024, 4097), (1040, 1024, 3072),
    (1040, 1024, 4000), (1920, 1632, 1000)])
def test_tile_lists_by_route(w, h, n):
    say(f"test_tile_lists_by_route {w}x{h} n={n}")
    cam = synth.make_camera(w, h)
    rng = np.random.default_rng(w + n)
    z = rng.uniform(1.5, 6.0, n)
    means = np.stack([(rng.uniform(0, w, n) - cam.cx) / cam.fx * z,
                      (rng.uniform(0, h, n) - cam.cy) / cam.fy * z, z], 1)
    px = np.exp(rng.uniform(0.0, 3.0, (n, 3)))
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()
    scene = (d(means), d(np.log(px * z[:, None] / cam.fx)), d(rng.normal(size=(n, 4))),
             d(rng.uniform(-2, 2, n)), d(rng.uniform(0, 1, (n, 3))))
    st = rtgs.Renderer(0, check="every").forward(scene, d(eye_view()), rcam(cam))
    dbg = st.stage()
    g = dbg["stage"]
    seen = st.visible.cpu().numpy().astype(bool)
    ranges, ids = binning.tile_lists(g[:, 0], g[:, 1], g[:, 7], g[:, 8], g[:, 6], seen, w, h)
    assert np.array_equal(dbg["ranges"], ranges)
    assert np.array_equal(dbg["ids"], ids)
