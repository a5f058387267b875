"""Saved fragments: images and gradients bitwise those of the saved per-pixel
state, with lists that end inside a group of four entries, with a step and past
one, on the pixel grid, on downsampled frames, and with lanes by previous work."""
import numpy as np
import pytest
import torch

from paper_2510_06644_amd import rtgs, synth
from tests.gpu_util import eye_view, rcam, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 3, 4, 15, 16, 18, 63, 65, 2000])
@pytest.mark.parametrize("j", [0, 2, 3])
@pytest.mark.parametrize("balance", [False, True])
def test_fragments_equal_the_saved_state(n, j, balance):
    say(f"test_fragments n={n} j={j} balance={balance}")
    w, h = 75, 53
    cam = synth.make_camera(w, h)
    rng = np.random.default_rng(n)
    z = rng.uniform(1.5, 6.0, n)
    means = np.stack([(rng.uniform(0, w, n) - cam.cx) / cam.fx * z,
                      (rng.uniform(0, h, n) - cam.cy) / cam.fy * z, z], 1)
    px = np.exp(rng.uniform(np.log(2.0), np.log(25.0), (n, 3)))
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()
    # (some of them clamped at 0.99)
    scene = (d(means), d(np.log(px * z[:, None] / cam.fx)), d(rng.normal(size=(n, 4))),
             d(rng.uniform(-3, 7, n)), d(rng.uniform(0, 1, (n, 3))))
    view, rc = d(eye_view()), rcam(cam)
    up = [d(rng.normal(size=(3, h, w))), d(rng.normal(size=(h, w))), d(rng.normal(size=(h, w)))]
    kw = dict(sample_log2=j)
    mask = None
    if j:
        mask = torch.empty(h, w, dtype=torch.uint8, device="cuda")
        rtgs.downsample_mask(d(rng.uniform(size=(h, w))), j, mask)
        kw["pixel_mask"] = mask
    if balance:
        kw.update(balance=True,
                  lane_work=torch.from_numpy(rng.integers(0, 40, (h, w)).astype(np.uint16)).cuda())
    r = rtgs.Renderer(0, check="every")
    a = r.forward(scene, view, rc, **kw)
    b = r.forward(scene, view, rc, save_fragments=True, **kw)
    for k in ("color", "depth", "alpha", "final_T", "last_idx"):
        assert torch.equal(getattr(a, k), getattr(b, k)), k
    for map_grads in (True, False):
        ga, gb = (r.backward(scene, view, rc, st, *up, map_grads=map_grads, pixel_mask=mask)
                  for st in (a, b))
        for k in ga:
            assert torch.equal(ga[k], gb[k]), k
