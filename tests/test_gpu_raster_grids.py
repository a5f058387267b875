"""The rasterizers' codes by sample grid: a masked frame with one sample a block
of pixels (8, 16 or any number of columns a quadrant) gives bitwise the image of
the same masked frame without blocks, whose tiles and lists differ, and its
gradients up to the order of summation (within GRAD_TOL of their norm, the bound
of each Gaussian's gradient against the oracle); with few and with many tiles, for all gradients and for the pose's, and
with groups of fewer than 8, exactly 8 and more entries a quadrant."""
import numpy as np
import pytest
import torch

from paper_2510_06644_amd import rtgs, synth
from tests.gpu_util import GRAD_TOL, eye_view, norm_err, rcam, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,n", [(97, 71, 5), (97, 71, 3000), (640, 521, 6000)])
@pytest.mark.parametrize("j", [1, 2, 3, 4])
@pytest.mark.parametrize("map_grads", [False, True])
def test_sample_blocks_match_the_pixel_grid(w, h, n, j, map_grads):
    say(f"test_sample_blocks {w}x{h} n={n} j={j} map={map_grads}")
    cam = synth.make_camera(w, h)
    rng = np.random.default_rng(n + j)
    z = rng.uniform(1.5, 6.0, n)
    means = np.stack([(rng.uniform(0, w, n) - cam.cx) / cam.fx * z,
                      (rng.uniform(0, h, n) - cam.cy) / cam.fy * z, z], 1)
    px = np.exp(rng.uniform(np.log(0.4), np.log(25.0), (n, 3)))       # scales in pixels
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()
    scene = (d(means), d(np.log(px * z[:, None] / cam.fx)), d(rng.normal(size=(n, 4))),
             d(rng.uniform(-2, 2, n)), d(rng.uniform(0, 1, (n, 3))))
    view, rc = d(eye_view()), rcam(cam)
    r = rtgs.Renderer(0, check="every")
    full = r.forward(scene, view, rc)
    mask = torch.empty(h, w, dtype=torch.uint8, device="cuda")
    rtgs.downsample_mask(full.final_T, j, mask)
    up = [d(rng.normal(size=(3, h, w))), d(rng.normal(size=(h, w))), d(rng.normal(size=(h, w)))]
    got = []
    for sub in (j, 0):
        st = r.forward(scene, view, rc, pixel_mask=mask, sample_log2=sub)
        g = r.backward(scene, view, rc, st, *up, pose=True, map_grads=map_grads, pixel_mask=mask)
        got.append((st, g))
    (a, ga), (b, gb) = got
    for k in ("color", "depth", "alpha", "final_T"):
        assert torch.equal(getattr(a, k), getattr(b, k)), k
    for k in gb:
        e = norm_err(ga[k].cpu().numpy(), gb[k].cpu().numpy())
        say(f"  {k}: {e:.2e}")
        assert e < GRAD_TOL, k
